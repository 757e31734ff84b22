// conv_any.hip -- a convolution stage of any supported filter (1..11),
// stride (1..4), padding and channel counts on the matrix cores, bf16 or
// fp32 (folded batch-norm scale/bias, activation, optional fused 2x2/2
// max-pool): the layers that the kernels for "same" 1x1 and 3x3 convolutions
// with whole channel chunks do not take.
//
// GEMM: M = the tile's computed output pixels, N = output channels, K = the
// filter window in KRSC order, cut into 16-byte pieces (8 bf16 or 4 fp32).
// Two forms of K:
//   - whole pieces (GATHER = false, c_in a multiple of a piece): a piece lies
//     in one filter tap; it is fetched with buffer_load_dwordx4 ... lds
//     straight into the LDS ring, each lane keeping the tap and channel of its
//     piece and stepping them from stage to stage;
//   - ragged channels (GATHER = true: more of them than fit the LDS of
//     conv_thin.hip): the f * c_in values of one filter row are one contiguous
//     run of the NHWC input, and of the KRSC weights, so K runs over the f rows,
//     each padded to whole pieces.  A lane fetches the values of its piece one
//     by one (their place need not be aligned), packs them and writes the piece
//     to LDS.
// A value outside the image, past the end of K, past the tile's last pixel or
// past c_out is fetched at an offset with bit 31 set, past the buffer
// descriptor's range, and reads zero.
//
// Work split: BM pixels x BN channels per workgroup, KG groups of four waves
// (2 x 2 over the block); group g takes the 128-byte part g of every K
// stage, so a long K with few pixels runs in nstage / KG steps, and the
// groups' sums meet in LDS at the end.  Part p of K (128 bytes) belongs to
// partial sum p mod 4 whatever KG is (a group keeps 4 / KG of them), and the four
// are added in order: the block and the K groups, which follow the size of the
// launch, change no bit of a result.  These layers are small (a strided
// 3x3 on a 56x50 tile has 700 pixels): what bounds a launch is the chain of
// K steps of one workgroup and how many compute units have one, not the
// matrix cores, hence the small blocks and the K groups (choose_any in
// run.cpp).  Measured against one thread per output pixel on the vector ALUs,
// which these layers ran on before (strided stem on 224x200, four frames,
// bf16): 3x3/2 32->64 1389 -> under 9 us, 5x5 64->64 8774 -> under 9 us.  The
// four partial sums cost 0.7 % (528 layers and batches, 6 % at most).
//
// Requires byte offsets below 2^31 within a frame's source buffer and within
// the weights (checked by the host); a fused pool needs even tile origins
// and extents.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "kernel_args.h"

namespace mafat {
namespace {

template <int DT, int BM, int BN, int KG, bool POOL, bool GATHER>
__global__ __launch_bounds__(256 * KG) void conv_any_kernel(const StageArgs a) {
  if (__builtin_expect(blockIdx.y != 0, 0)) {  // the second grid row: carried band copies (row reuse)
    carried_copies();
    return;
  }
  using T = typename Elt<DT>::T;
  constexpr int ESZ = static_cast<int>(sizeof(T));
  constexpr int EPV = 16 / ESZ;                // values per 16-byte piece
  constexpr int NS = GATHER ? 2 : 3;           // ring slots
  constexpr int PART = (BM + BN) * 128;        // one K group's part of a slot (128 bytes per row)
  constexpr int SLOT = KG * PART;
  constexpr int APW = BM / 32, BPW = BN / 32;  // pieces per thread and stage (32 rows x 8 pieces per group and pass)
  constexpr int LPS = APW + BPW;
  constexpr int WM = BM / 2, WN = BN / 2, MT = WM / 16, NT = WN / 16;
  constexpr int RSB = BN * ESZ + 16;           // LDS bytes per staged output row
  constexpr int NPXO = POOL ? BM / 4 : BM;
  constexpr int NP = 4 / KG;                   // partial sums of a group
  static_assert(KG * NP == 4, "four partial sums");
  static_assert(APW >= 1 && BPW >= 1 && APW * 32 == BM && BPW * 32 == BN, "block shape");
  static_assert(NPXO * RSB <= NS * SLOT && (KG - 1) * NP * BM * BN * 4 <= NS * SLOT, "epilogue fits in the ring");
  __shared__ __align__(1024) unsigned char smem[NS * SLOT];

  KTile tl;
  const BlockPos bp = decode_block(a, &tl);
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, wq = wave & 3, wm = wq >> 1, wn = wq & 1;
  const int M = tl.ch * tl.cw, m0 = bp.mb * BM, n0 = bp.nb * BN;
  const int cin = a.cin, cout = a.cout, f = a.f, st = a.s, pd = a.p, sw = tl.sw;
  const int K = f * f * cin;
  const int64_t sbase = bp.frame * a.src_fstride + tl.src_off;
  T* dst = static_cast<T*>(a.dst) + bp.frame * a.dst_fstride + tl.dst_off;
  const __amdgpu_buffer_rsrc_t rsa =
      make_rsrc(static_cast<const T*>(a.src) + sbase, static_cast<unsigned>((a.src_fstride - tl.src_off) * ESZ));
  const __amdgpu_buffer_rsrc_t rsb = make_rsrc(a.w, static_cast<unsigned>(cout * K * ESZ));

  // K in runs of `run` pieces: the taps (whole pieces), or the filter rows
  // (ragged channels).
  const int run = GATHER ? (f * cin + EPV - 1) / EPV : cin / EPV;
  const int nrun = GATHER ? f : f * f;
  const int nstage = (run * nrun + 8 * KG - 1) / (8 * KG);
  const unsigned finv = 65536u / static_cast<unsigned>(f) + 1u;  // tap / f = tap * finv >> 16 (tap < 256, f <= 11)

  // This lane's pieces: rows wq * 8 + (lane >> 3) + 32 k of the A and the B
  // part, piece cg of each stage's 8 of this group (LDS position lane & 7,
  // swizzled by the row so that fragment reads of 16 rows spread over the
  // banks).  (kr, kc): run and piece in it of the next stage to load.
  const int lrow = lane >> 3, cg = (lane & 7) ^ lrow;
  int piece = grp * 8 + cg;                          // index of the piece in K
  int kr = piece / run, kc = piece - kr * run;
  const int step_r = (8 * KG) / run, step_c = 8 * KG - step_r * run;
  int py[APW], px[APW];  // top left input pixel of the row's window (whether in the image or not)
  bool pok[APW];
#pragma unroll
  for (int k = 0; k < APW; ++k) {
    const int m = m0 + wq * 8 + lrow + 32 * k;
    int oy, ox;
    row_pixel<POOL>(tl, m < M ? m : 0, &oy, &ox);
    py[k] = oy * st - pd;
    px[k] = ox * st - pd;
    pok[k] = m < M;
  }
  auto advance = [&]() {
    piece += 8 * KG;
    kc += step_c;
    kr += step_r;
    if (kc >= run) { kc -= run; ++kr; }
  };

  // Fragment reads: row (l & 15) of a 16-row fragment, piece 4 h + (l >> 4).
  int rd_a[2], rd_b[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int pos = ((h * 4 + (lane >> 4)) ^ (lane & 7)) * 16;
    rd_a[h] = grp * PART + (wm * WM + (lane & 15)) * 128 + pos;
    rd_b[h] = grp * PART + (BM + wn * WN + (lane & 15)) * 128 + pos;
  }
  f32x4 part[NP][NT][MT];
#pragma unroll
  for (int u = 0; u < NP; ++u)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) part[u][j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int slot, int u) {  // into partial sum u of this group's
    const unsigned char* sp = smem + slot * SLOT;
    u32x4 af[2][MT], bfr[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < MT; ++i) af[h][i] = *reinterpret_cast<const u32x4*>(sp + rd_a[h] + i * 16 * 128);
#pragma unroll
      for (int j = 0; j < NT; ++j) bfr[h][j] = *reinterpret_cast<const u32x4*>(sp + rd_b[h] + j * 16 * 128);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          if constexpr (POOL) mma<DT>(part[u][j][i], af[h][i], bfr[h][j]);
          else mma<DT>(part[u][j][i], bfr[h][j], af[h][i]);
        }
  };

  if constexpr (!GATHER) {
    auto issue = [&](int slot) {
      unsigned char* sp = smem + slot * SLOT + grp * PART + wq * 8 * 128;
      const int ky = static_cast<int>((static_cast<unsigned>(kr) * finv) >> 16), kx = kr - ky * f;
      const bool kok = kr < nrun;
#pragma unroll
      for (int k = 0; k < APW; ++k) {
        const int iy = py[k] + ky, ix = px[k] + kx;
        const bool ok = kok && pok[k] && static_cast<unsigned>(iy) < static_cast<unsigned>(a.in_h) &&
                        static_cast<unsigned>(ix) < static_cast<unsigned>(a.in_w);
        const unsigned off = static_cast<unsigned>(((iy - tl.sy0) * sw + (ix - tl.sx0)) * cin * ESZ + kc * 16);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsa, (lds_ptr_t)(sp + k * 32 * 128), 16,
                                                 static_cast<int>(ok ? off : 0x80000000u), 0, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < BPW; ++k) {
        const int co = n0 + wq * 8 + lrow + 32 * k;
        const bool ok = kok && co < cout;
        const unsigned off = static_cast<unsigned>(co * K * ESZ + piece * 16);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsb, (lds_ptr_t)(sp + (BM + k * 32) * 128), 16,
                                                 static_cast<int>(ok ? off : 0x80000000u), 0, 0, 0);
      }
      advance();
    };
#pragma unroll
    for (int p = 0; p < NS - 1; ++p)
      if (p < nstage) issue(p);
    int slot = 0;
    for (int s0 = 0; s0 < nstage; s0 += NP) {
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int s = s0 + u;
        if (s >= nstage) break;
        wait_stage<LPS, NS - 2>(nstage - 1 - s);
        wg_barrier();  // stage s is in LDS; every wave is done reading the slot before it
        if (s + NS - 1 < nstage) issue(slot == 0 ? NS - 1 : slot - 1);
        compute(slot, u);
        slot = (slot == NS - 1) ? 0 : slot + 1;
      }
    }
  } else {
    // Values of this lane's pieces of the next stage, into registers.
    u32x4 ra[APW], rb[BPW];
    auto load_piece = [&](__amdgpu_buffer_rsrc_t rs, unsigned base, int e_lo, int e_hi) {
      u32x4 v;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if constexpr (DT == MAFAT_BF16) {
          const int e = kc * EPV + 2 * w;
          const unsigned lo = __builtin_amdgcn_raw_buffer_load_b16(
              rs, static_cast<int>(e >= e_lo && e < e_hi ? base + static_cast<unsigned>(e * 2) : 0x80000000u), 0, 0);
          const unsigned hi = __builtin_amdgcn_raw_buffer_load_b16(
              rs, static_cast<int>(e + 1 >= e_lo && e + 1 < e_hi ? base + static_cast<unsigned>(e * 2 + 2) : 0x80000000u),
              0, 0);
          v[w] = (lo & 0xffffu) | (hi << 16);
        } else {
          const int e = kc * EPV + w;
          v[w] = __builtin_amdgcn_raw_buffer_load_b32(
              rs, static_cast<int>(e >= e_lo && e < e_hi ? base + static_cast<unsigned>(e * 4) : 0x80000000u), 0, 0);
        }
      }
      return v;
    };
    auto load = [&]() {
      const bool kok = kr < nrun;
      const int fc = f * cin;
#pragma unroll
      for (int k = 0; k < APW; ++k) {
        // the values of filter row kr inside the image: [e_lo, e_hi) of f * c_in
        const int iy = py[k] + kr;
        const bool ok = kok && pok[k] && static_cast<unsigned>(iy) < static_cast<unsigned>(a.in_h);
        const int e_lo = max(-px[k], 0) * cin, e_hi = ok ? min(fc, (a.in_w - px[k]) * cin) : 0;
        ra[k] = load_piece(rsa, static_cast<unsigned>(((iy - tl.sy0) * sw + (px[k] - tl.sx0)) * cin * ESZ), e_lo, e_hi);
      }
#pragma unroll
      for (int k = 0; k < BPW; ++k) {
        const int co = n0 + wq * 8 + lrow + 32 * k;
        rb[k] = load_piece(rsb, static_cast<unsigned>((co * K + kr * fc) * ESZ), 0, (kok && co < cout) ? fc : 0);
      }
      advance();
    };
    auto commit = [&](int slot) {
      unsigned char* sp = smem + slot * SLOT + grp * PART + (wq * 8 + lrow) * 128 + (lane & 7) * 16;
#pragma unroll
      for (int k = 0; k < APW; ++k) *reinterpret_cast<u32x4*>(sp + k * 32 * 128) = ra[k];
#pragma unroll
      for (int k = 0; k < BPW; ++k) *reinterpret_cast<u32x4*>(sp + (BM + k * 32) * 128) = rb[k];
    };
    load();
    commit(0);
    for (int s0 = 0; s0 < nstage; s0 += NP) {
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int s = s0 + u;
        if (s >= nstage) break;
        __syncthreads();  // stage s is in LDS; every wave is done reading the other slot
        if (s + 1 < nstage) load();
        compute(s & 1, u);
        if (s + 1 < nstage) commit((s + 1) & 1);
      }
    }
  }

  // The partial sums meet: group 0 adds the four in order.  Partial sum p is
  // number p / KG of group p % KG.
  __syncthreads();  // every wave is done reading the ring
  f32x4 acc[NT][MT];
  f32x4* sx = reinterpret_cast<f32x4*>(smem);  // [(group - 1) * NP + number][wave of the group][NT][MT][64 lanes]
  if constexpr (KG > 1) {
    if (grp > 0) {
#pragma unroll
      for (int u = 0; u < NP; ++u)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int i = 0; i < MT; ++i)
            sx[(((((grp - 1) * NP + u) * 4 + wq) * NT + j) * MT + i) * 64 + lane] = part[u][j][i];
    }
    __syncthreads();
  }
  if (grp == 0) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        acc[j][i] = part[0][j][i];
#pragma unroll
        for (int p = 1; p < 4; ++p)
          acc[j][i] += p % KG == 0 ? part[p / KG][j][i]
                                   : sx[((((p % KG - 1) * NP + p / KG) * 4 + wq) * NT + j) * MT * 64 + i * 64 + lane];
      }
  }
  if constexpr (KG > 1) __syncthreads();

  // Epilogue (group 0): scale, bias, the fused pool, activation; the block's
  // outputs are staged in LDS as rows of BN channels.
  const float slope = act_slope(a.act);
  if (grp == 0) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      float sc[4], bi[4];
#pragma unroll
      for (int r = 0; r < (POOL ? 1 : 4); ++r) {
        const int co = n0 + wn * WN + j * 16 + (POOL ? (lane & 15) : 4 * (lane >> 4) + r);
        sc[r] = a.scale[min(co, cout - 1)];
        bi[r] = a.bias[min(co, cout - 1)];
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if constexpr (POOL) {
          const int rl = wm * WM + i * 16 + 4 * (lane >> 4);  // first block row of this lane's window
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = fmaf(acc[j][i][r], sc[0], bi[0]);
          float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
          mx = fmaxf(mx, slope * mx);
          store1(reinterpret_cast<T*>(smem + (rl >> 2) * RSB) + wn * WN + j * 16 + (lane & 15), mx);
        } else {
          const int rl = wm * WM + i * 16 + (lane & 15);
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[r] = fmaf(acc[j][i][r], sc[r], bi[r]);
            v[r] = fmaxf(v[r], slope * v[r]);
          }
          store4<DT>(reinterpret_cast<T*>(smem + rl * RSB) + wn * WN + j * 16 + 4 * (lane >> 4), v);
        }
      }
    }
  }
  __syncthreads();
  // Out: 16 bytes per thread and step where pixels start at 16-byte
  // boundaries (c_out whole pieces), else value by value.
  const bool vec = cout % EPV == 0;
  const int per = vec ? BN / EPV : BN;  // stores per pixel row
  for (int e = tid; e < NPXO * per; e += 256 * KG) {
    const int p = e / per, k = e - p * per;
    const int m = m0 + (POOL ? 4 * p : p);
    const int c0 = n0 + (vec ? k * EPV : k);
    if (m < M && c0 < cout) {
      int oy, ox;
      row_pixel<POOL>(tl, m, &oy, &ox);
      if (POOL) { oy >>= 1; ox >>= 1; }
      T* o = dst + ((oy - tl.dy0) * tl.dw + (ox - tl.dx0)) * cout + c0;
      const unsigned char* s = smem + p * RSB + (vec ? k * 16 : k * ESZ);
      if (vec) *reinterpret_cast<u32x4*>(o) = *reinterpret_cast<const u32x4*>(s);
      else *o = *reinterpret_cast<const T*>(s);
    }
  }
}

template <int DT, bool POOL, bool GATHER>
hipError_t launch_any(const MfmaShape& sh, const StageArgs& args, hipStream_t stream, LaunchEvents ev) {
  const dim3 grid(static_cast<unsigned>(args.total_blocks), args.copy_blocks > 0 ? 2u : 1u);
#define MAFAT_ANY(bm_, bn_, kg_)                                                                           \
  if (sh.bm == (bm_) && sh.bn == (bn_) && sh.kg == (kg_)) {                                                \
    hipExtLaunchKernelGGL((conv_any_kernel<DT, bm_, bn_, kg_, POOL, GATHER>), grid, dim3(256 * (kg_)), 0,  \
                          stream, ev.start, ev.stop, 0, args);                                             \
    return hipGetLastError();                                                                              \
  }
  MAFAT_ANY_SHAPES
#undef MAFAT_ANY
  return hipErrorInvalidValue;
}

template <int DT>
hipError_t launch_any_dt(bool pool, const MfmaShape& sh, const StageArgs& args, hipStream_t stream, LaunchEvents ev) {
  const bool gather = args.cin % (DT == MAFAT_BF16 ? 8 : 4) != 0;
  if (pool) return gather ? launch_any<DT, true, true>(sh, args, stream, ev) : launch_any<DT, true, false>(sh, args, stream, ev);
  return gather ? launch_any<DT, false, true>(sh, args, stream, ev) : launch_any<DT, false, false>(sh, args, stream, ev);
}

}  // namespace

hipError_t launch_conv_any(int dtype, bool pool, const MfmaShape& shape, const StageArgs& args, hipStream_t stream,
                           LaunchEvents ev) {
  if (args.total_blocks <= 0) return hipSuccess;
  if (dtype == MAFAT_BF16) return launch_any_dt<MAFAT_BF16>(pool, shape, args, stream, ev);
  if (dtype == MAFAT_F32) return launch_any_dt<MAFAT_F32>(pool, shape, args, stream, ev);
  return hipErrorInvalidValue;
}

}  // namespace mafat
