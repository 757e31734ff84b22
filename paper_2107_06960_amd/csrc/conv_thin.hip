// conv_thin.hip -- a convolution stage whose input channels fill no 16-byte
// piece (an image's three), any filter, stride and padding, bf16 or fp32, on
// the matrix cores (folded batch-norm scale/bias, activation, optional fused
// 2x2/2 max-pool).
//
// A workgroup owns a BR x BC block of conv outputs of one tile and BN output
// channels.  Its input patch is staged in LDS once, as the rows of values it
// is in memory, and its weights (KRSC) as they are.  NHWC makes the f * c_in
// values that a filter row reads contiguous from any pixel on, in the patch
// and in the weights alike, so an operand is read at its place in either:
//   - fp32: K runs over the f f c_in values, four to an MFMA, a lane reading
//     one; a table gives each value's place in the patch;
//   - bf16: K runs over the filter rows, each cut into 8-value pieces, four to
//     an MFMA; a piece starts at any value, so a lane reads the five words
//     that hold it, shifts them and clears what lies past the filter row; a
//     table gives each piece's places and what it keeps.
//
// What bounds it: K is short (27 to 147 values), so a workgroup is its loads,
// one barrier, a few MFMAs per tile and its stores, and several workgroups
// share a compute unit.  In us a launch, before (3x3 in fp32 one thread per
// pixel or window on the vector ALUs, the others gathered value by value per
// output pixel) and now: 3->16 and pool on 64x64, four tiles, fp32 6.2 and 4.6;
// 3->64 on 131x97, two frames, fp32 10.1 and 7.2; 7x7/2 3->32 on 224x200, four
// frames, bf16 16.4 and 9.0, one frame, fp32 16.0 and 12.0; 3->32 and pool on
// 416x416, nine tiles, fp32 18.5 and 18.5 to 19.
//
// Requires byte offsets below 2^31 within a frame's source buffer and the
// patch, weights and table in kThinLds bytes (checked by the host); a fused
// pool needs even tile origins and extents.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "kernel_args.h"

namespace mafat {
namespace {

template <int DT, int BR, int BC, int BN, bool POOL>
__global__ __launch_bounds__(256) void conv_thin_kernel(const StageArgs a) {
  if (__builtin_expect(blockIdx.y != 0, 0)) {  // the second grid row: carried band copies (row reuse)
    carried_copies();
    return;
  }
  using T = typename Elt<DT>::T;
  constexpr int ESZ = static_cast<int>(sizeof(T));
  constexpr int BM = BR * BC, MT = BM / 64, NT = BN / 16;  // 4 waves, each BM / 4 pixels and all channels
  static_assert(MT * 64 == BM && BR % 2 == 0 && BC % 2 == 0, "block");
  extern __shared__ __align__(16) unsigned char smem[];

  KTile tl;
  const BlockPos bp = decode_block(a, &tl);
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cin = a.cin, cout = a.cout, f = a.f, st = a.s, pd = a.p;
  const ThinLayout L = thin_layout(BR, BC, BN, f, st, cin, ESZ);
  const int nbx = (tl.cw + BC - 1) / BC;
  const int bby = div_small(bp.mb, nbx), bbx = bp.mb - bby * nbx;
  const int by0 = tl.cy0 + bby * BR, bx0 = tl.cx0 + bbx * BC;  // block origin (conv outputs)
  const int n0 = bp.nb * BN;
  const int64_t sbase = bp.frame * a.src_fstride + tl.src_off;
  T* dst = static_cast<T*>(a.dst) + bp.frame * a.dst_fstride + tl.dst_off;
  const __amdgpu_buffer_rsrc_t rsa =
      make_rsrc(static_cast<const T*>(a.src) + sbase, static_cast<unsigned>((a.src_fstride - tl.src_off) * ESZ));

  auto load1 = [&](__amdgpu_buffer_rsrc_t rs, unsigned off) {
    if constexpr (DT == MAFAT_BF16) return static_cast<T>(__builtin_amdgcn_raw_buffer_load_b16(rs, static_cast<int>(off), 0, 0));
    else return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, static_cast<int>(off), 0, 0));
  };
  const int fc = f * cin, K = f * fc;
  // Weights of the block's channels, one contiguous run: 16-byte pieces, then
  // the values past the last whole one.  Rows past c_out stay unwritten: they
  // only reach outputs that are not stored.
  // Patch: input rows by0 * s - p .., columns bx0 * s - p ..; a thread keeps
  // its column (of values) and steps over rows, or the other way round where a
  // row is longer than the workgroup.  Zero outside the image and outside what
  // this tile's outputs read.
  // The first loads of both go out before any of them is waited for, and so
  // do the scale and bias: a workgroup is too short to hide them otherwise.
  constexpr int UW = 5, UP = 6;  // pieces and values in flight per thread
  const int bytes = min(BN, cout - n0) * K * ESZ, n16 = bytes / 16;
  const unsigned char* wsrc = static_cast<const unsigned char*>(a.w) + static_cast<int64_t>(n0) * K * ESZ;
  u32x4 wv[UW];
  auto load_w = [&](int e0) {
#pragma unroll
    for (int u = 0; u < UW; ++u)
      if (e0 + 256 * u < n16) wv[u] = *reinterpret_cast<const u32x4*>(wsrc + (e0 + 256 * u) * 16);
  };
  auto put_w = [&](int e0) {
#pragma unroll
    for (int u = 0; u < UW; ++u)
      if (e0 + 256 * u < n16) *reinterpret_cast<u32x4*>(smem + L.weights + (e0 + 256 * u) * 16) = wv[u];
  };
  const int iy0 = by0 * st - pd, ix0 = bx0 * st - pd;
  const int ylo = max(tl.cy0 * st - pd, 0), yhi = min((tl.cy0 + tl.ch - 1) * st - pd + f, a.in_h);
  const int xlo = max(tl.cx0 * st - pd, 0), xhi = min((tl.cx0 + tl.cw - 1) * st - pd + f, a.in_w);
  const int e_lo = (xlo - ix0) * cin, e_hi = (xhi - ix0) * cin;  // values of a patch row that are read
  const int nr = max(256 / L.row_vals, 1);                      // rows per pass
  const int r0 = L.row_vals < 256 ? div_small(tid, L.row_vals) : 0;
  const int c0 = r0 < nr ? tid - r0 * L.row_vals : L.row_vals;  // threads past the last row of a pass: none
  T pv[UP];
  auto load_p = [&](int c, int r) {
    const bool cok = c >= e_lo && c < e_hi && c < L.row_vals;
#pragma unroll
    for (int u = 0; u < UP; ++u) {
      const int iy = iy0 + r + u * nr;
      const bool ok = cok && r + u * nr < L.rows && iy >= ylo && iy < yhi;
      pv[u] = load1(rsa, ok ? static_cast<unsigned>((((iy - tl.sy0) * tl.sw + (ix0 - tl.sx0)) * cin + c) * ESZ) : 0x80000000u);
    }
  };
  auto put_p = [&](int c, int r) {
#pragma unroll
    for (int u = 0; u < UP; ++u)
      if (c < L.row_vals && r + u * nr < L.rows)
        *reinterpret_cast<T*>(smem + L.patch + (r + u * nr) * L.row_bytes + c * ESZ) = pv[u];
  };
  load_w(tid);
  load_p(c0, r0);
  float sc[NT][4], bi[NT][4];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int r = 0; r < (POOL ? 1 : 4); ++r) {
      const int co = min(n0 + j * 16 + (POOL ? (lane & 15) : 4 * (lane >> 4) + r), cout - 1);
      sc[j][r] = a.scale[co];
      bi[j][r] = a.bias[co];
    }
  // Table.  fp32: value k's place relative to a pixel's window.  bf16: the
  // bits piece P keeps, its place in the window and in a weight row.
  for (int e = tid; e < 4 * L.steps; e += 256) {
    if constexpr (DT == MAFAT_BF16) {
      const int ky = div_small(e, L.run), k0 = (e - ky * L.run) * 8;
      const int keep = ky < f ? min(fc - k0, 8) : 0;  // values
      u32x4 m;
#pragma unroll
      for (int w = 0; w < 4; ++w) m[w] = keep >= 2 * w + 2 ? ~0u : keep == 2 * w + 1 ? 0xffffu : 0u;
      *reinterpret_cast<u32x4*>(smem + e * 32) = m;
      *reinterpret_cast<int*>(smem + e * 32 + 16) = ky < f ? ky * L.row_bytes + k0 * 2 : 0;
      *reinterpret_cast<int*>(smem + e * 32 + 20) = ky < f ? (ky * fc + k0) * 2 : 0;
    } else {
      const int ky = div_small(e, fc);
      *reinterpret_cast<int*>(smem + e * 4) = e < K ? ky * L.row_bytes + (e - ky * fc) * 4 : 0;
    }
  }
  put_w(tid);
  for (int e0 = tid + 256 * UW; e0 < n16; e0 += 256 * UW) {
    load_w(e0);
    put_w(e0);
  }
  const int tail = n16 * 16 + tid * ESZ;
  if (tail < bytes) *reinterpret_cast<T*>(smem + L.weights + tail) = *reinterpret_cast<const T*>(wsrc + tail);
  put_p(c0, r0);
  for (int c = c0; c < L.row_vals; c += 256)
    for (int r = c == c0 ? r0 + nr * UP : r0; r < L.rows; r += nr * UP) {
      load_p(c, r);
      put_p(c, r);
    }
  __syncthreads();

  const int q = lane >> 4, l15 = lane & 15;
  int xb[MT], wb[NT];  // places of this lane's windows and weight rows
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int y, x;
    block_pixel<BC>(wave * (BM / 4) + i * 16 + l15, &y, &x);
    xb[i] = L.patch + y * st * L.row_bytes + x * st * cin * ESZ;
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) wb[j] = L.weights + (j * 16 + l15) * K * ESZ;
  f32x4 acc[NT][MT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (DT == MAFAT_BF16) {
    auto piece = [&](int at, const u32x4& keep) {  // the 8 values at byte `at`
      const unsigned* p = reinterpret_cast<const unsigned*>(smem + (at & ~3));
      const unsigned d0 = p[0], d1 = p[1], d2 = p[2], d3 = p[3], d4 = p[4];
      const unsigned sh = static_cast<unsigned>(at & 2) * 8u;
      return u32x4{__builtin_amdgcn_alignbit(d1, d0, sh), __builtin_amdgcn_alignbit(d2, d1, sh),
                   __builtin_amdgcn_alignbit(d3, d2, sh), __builtin_amdgcn_alignbit(d4, d3, sh)} & keep;
    };
    for (int s = 0; s < L.steps; ++s) {
      const unsigned char* t = smem + (4 * s + q) * 32;
      const u32x4 keep = *reinterpret_cast<const u32x4*>(t);
      const int xo = *reinterpret_cast<const int*>(t + 16), wo = *reinterpret_cast<const int*>(t + 20);
      u32x4 wf[NT], xf[MT];
#pragma unroll
      for (int j = 0; j < NT; ++j) wf[j] = piece(wb[j] + wo, keep);
#pragma unroll
      for (int i = 0; i < MT; ++i) xf[i] = piece(xb[i] + xo, keep);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          if constexpr (POOL) mma<DT>(acc[j][i], xf[i], wf[j]);
          else mma<DT>(acc[j][i], wf[j], xf[i]);
        }
    }
  } else {
    // U steps at a time, so that their reads (the table's, then the patch's)
    // are in flight together; steps and values past K take zeros.
    constexpr int U = 4;
    for (int s0 = 0; s0 < L.steps; s0 += U) {
      int xo[U];
      float wf[U][NT], xf[U][MT];
#pragma unroll
      for (int u = 0; u < U; ++u) xo[u] = *reinterpret_cast<const int*>(smem + min(4 * (s0 + u) + q, K - 1) * 4);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = 4 * (s0 + u) + q;
#pragma unroll
        for (int j = 0; j < NT; ++j) wf[u][j] = *reinterpret_cast<const float*>(smem + wb[j] + min(k, K - 1) * 4);
#pragma unroll
        for (int i = 0; i < MT; ++i) xf[u][i] = *reinterpret_cast<const float*>(smem + xb[i] + xo[u]);
      }
      if (4 * (s0 + U) > K) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = 4 * (s0 + u) + q < K;
#pragma unroll
          for (int j = 0; j < NT; ++j) wf[u][j] = in ? wf[u][j] : 0.f;
#pragma unroll
          for (int i = 0; i < MT; ++i) xf[u][i] = in ? xf[u][i] : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= L.steps) break;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[j][i] = POOL ? __builtin_amdgcn_mfma_f32_16x16x4f32(xf[u][i], wf[u][j], acc[j][i], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_16x16x4f32(wf[u][j], xf[u][i], acc[j][i], 0, 0, 0);
      }
    }
  }

  // Epilogue, from registers: without a pool a lane holds 4 consecutive
  // channels of one pixel, with one a channel of one window.
  const float slope = act_slope(a.act);
  const int vy = tl.cy0 + tl.ch - by0, vx = tl.cx0 + tl.cw - bx0;  // valid extent of this block
  const bool vec = (cout & 3) == 0;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int co = n0 + j * 16 + (POOL ? l15 : 4 * q);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      int y, x;
      block_pixel<BC>(wave * (BM / 4) + i * 16 + (POOL ? 4 * q : l15), &y, &x);
      if (y >= vy || x >= vx || co >= cout) continue;
      const int oy = POOL ? (by0 + y) >> 1 : by0 + y, ox = POOL ? (bx0 + x) >> 1 : bx0 + x;
      T* o = dst + ((oy - tl.dy0) * tl.dw + (ox - tl.dx0)) * cout + co;
      float v[4];
      if constexpr (POOL) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(acc[j][i][r], sc[j][0], bi[j][0]);
        const float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
        store1(o, fmaxf(mx, slope * mx));
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = fmaf(acc[j][i][r], sc[j][r], bi[j][r]);
          v[r] = fmaxf(v[r], slope * v[r]);
        }
        if (vec) {
          store4<DT>(o, v);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (co + r < cout) store1(o + r, v[r]);
        }
      }
    }
  }
}

template <int DT, bool POOL>
hipError_t launch_thin(const MfmaShape& sh, const StageArgs& args, hipStream_t stream, LaunchEvents ev) {
  const dim3 grid(static_cast<unsigned>(args.total_blocks), args.copy_blocks > 0 ? 2u : 1u);
  const ThinLayout L = thin_layout(sh.br, sh.bc, sh.bn, args.f, args.s, args.cin, DT == MAFAT_BF16 ? 2 : 4);
  if (L.total > kThinLds) return hipErrorInvalidValue;
#define MAFAT_THIN(br_, bc_, bn_)                                                                            \
  if (sh.br == (br_) && sh.bc == (bc_) && sh.bn == (bn_)) {                                                  \
    hipExtLaunchKernelGGL((conv_thin_kernel<DT, br_, bc_, bn_, POOL>), grid, dim3(256),                      \
                          static_cast<unsigned>(L.total), stream, ev.start, ev.stop, 0, args);               \
    return hipGetLastError();                                                                                \
  }
  MAFAT_THIN_SHAPES
#undef MAFAT_THIN
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_conv_thin(int dtype, bool pool, const MfmaShape& shape, const StageArgs& args, hipStream_t stream,
                            LaunchEvents ev) {
  if (args.total_blocks <= 0) return hipSuccess;
  if (dtype == MAFAT_BF16)
    return pool ? launch_thin<MAFAT_BF16, true>(shape, args, stream, ev)
                : launch_thin<MAFAT_BF16, false>(shape, args, stream, ev);
  if (dtype == MAFAT_F32)
    return pool ? launch_thin<MAFAT_F32, true>(shape, args, stream, ev)
                : launch_thin<MAFAT_F32, false>(shape, args, stream, ev);
  return hipErrorInvalidValue;
}

}  // namespace mafat
