// conv_ring.hip -- bf16 1x1 convolution stage (stride 1, folded batch-norm
// scale/bias, activation, optional fused 2x2/2 max-pool) as a GEMM on the
// matrix cores, with its operands streamed from global memory straight into
// a ring of LDS stage slots.
//
// GEMM: M = the tile's computed output pixels, N = output channels, K =
// c_in.  One K stage is 64 channels = 128 bytes of every A row (pixel) and B
// row (output channel); where c_in is an odd multiple of 32 the last stage's
// second half is zeros.
//
// Data movement (per workgroup, BM pixels x BN channels):
//   - A ring of NS slots in LDS, each holding one K stage of the BM + BN
//     rows (128 bytes per row).  Stage s lives in slot s % NS.
//   - Each thread fetches 16-byte pieces with buffer_load_dwordx4 ... lds:
//     the data goes from L2/HBM directly into LDS (no VGPR staging), 64
//     lanes filling 1 KiB = 8 rows of one slot per instruction.  Lane l
//     writes row (l >> 3), 16-byte position (l & 7) of its 8-row group and
//     fetches the global 16-byte chunk (l & 7) ^ (l >> 3) of that row: an
//     XOR swizzle of the chunk position by the row, so the fragment reads of
//     16 consecutive rows at one K offset spread over all LDS banks.
//   - A pixel past the tile's last row, a weight row past c_out and the half
//     stage past the last channel are fetched at an offset with bit 31 set,
//     past the buffer descriptor's range, and the range check returns zeros.
//   - Loads run NS - 1 stages ahead of the MFMAs.  Iteration s waits (an
//     explicit s_waitcnt vmcnt) until this thread's loads of stage s have
//     landed, meets the other waves at a barrier (then stage s is complete
//     in LDS and every wave is done reading slot (s - 1) % NS), issues the
//     loads of stage s + NS - 1 into that freed slot, reads its MFMA
//     fragments of stage s and runs the MFMAs.
// Compute: waves in a WGM x WGN arrangement over the block, each owning a
// (BM/WGM) x (BN/WGN) tile of 16x16 accumulators, v_mfma_f32_16x16x32_bf16.
// Epilogue: without a pool the weights are the MFMA's A operand, so a lane
// holds 4 consecutive channels of one pixel; with a fused pool the pixels
// are, quad-ordered, so a lane's 4 accumulator rows are one 2x2 window,
// reduced in the lane.  The block's outputs are staged in LDS as rows of BN
// channels and leave as 16-byte stores.  The first stage's weight rows are
// issued while the tile table is being decoded.
//
// Bounds: small launches by fixed cost and the chain of K steps (512->256 on
// 38x38: 4.75 us with 32x64 blocks), large ones by the L2->LDS rate (eight
// frames: 8.3 us with 64x64 blocks).  Offsets of a K step are one addition; a
// form that also walked filter taps and split K between two wave groups took
// 5.3 and 12.5 us (with its 32x64 blocks) on the same two.
//
// Requires c_in % 32 == 0, c_out % 16 == 0, byte offsets below 2^31 within
// a frame's source buffer and within the weights (checked by the host).
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "kernel_args.h"

namespace mafat {
#ifdef MAFAT_TUNING
// Tuning builds only: phase timestamps (wall clock, 100 MHz) of three
// workgroups (the first, the middle and the last of the grid).
__device__ long long g_ring_trace[3][64];
MAFAT_WG_TRACE_DECL(g_wg_ring)
#define MAFAT_RTRACE(slot_)                                                                      \
  do {                                                                                           \
    if (threadIdx.x == 0 && (slot_) < 64 &&                                                      \
        (blockIdx.x == 0 || blockIdx.x == a.total_blocks / 2 || blockIdx.x == a.total_blocks - 1))         \
      g_ring_trace[blockIdx.x == 0 ? 0 : (blockIdx.x == a.total_blocks - 1 ? 2 : 1)][(slot_)] =       \
          wall_clock64();                                                                        \
  } while (0)
#else
#define MAFAT_RTRACE(slot_) do {} while (0)
#endif
namespace {

template <int BM, int BN, int WGM, int WGN, int NS, bool POOL>
__global__ __launch_bounds__(64 * WGM * WGN) void conv_ring_kernel(const StageArgs a) {
  if (__builtin_expect(blockIdx.y != 0, 0)) {  // the second grid row: carried band copies (row reuse)
    carried_copies();
    return;
  }
  constexpr int NWAVE = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN, MT = WM / 16, NT = WN / 16;
  constexpr int ROWB = 128;                 // bytes of one row per K stage
  constexpr int SLOT = (BM + BN) * ROWB;    // bytes of one ring slot
  constexpr int APW = BM / (8 * NWAVE);     // A load instructions per wave per stage
  constexpr int BPW = BN / (8 * NWAVE);     // B load instructions per wave per stage
  constexpr int LPS = APW + BPW;            // loads per thread per stage
  constexpr int NH = 2;                     // 64-byte halves of a stage (one MFMA's K each)
  static_assert(MT >= 1 && NT >= 1 && MT * 16 == WM && NT * 16 == WN, "wave tile");
  static_assert(APW >= 1 && BPW >= 1 && APW * 8 * NWAVE == BM && BPW * 8 * NWAVE == BN, "load split");
  static_assert(NS >= 2 && NS <= 8 && (NS - 2) * LPS <= 63, "ring depth");
  __shared__ __align__(1024) unsigned char smem[NS * SLOT];

  MAFAT_RTRACE(0);
  MAFAT_WG_MARK(g_wg_ring, 0);
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cin = a.cin, cout = a.cout;
  const int nstage = (cin + 63) >> 6;
  const __amdgpu_buffer_rsrc_t rsb = make_rsrc(a.w, static_cast<unsigned>(cout * cin * 2));
  // This lane's loads: row (lane >> 3) of 8-row group (k * NWAVE + wave) of
  // the A rows (k < APW) and of the B rows (k < BPW); global 16-byte chunk
  // cg of the 128-byte stage row.
  const int lrow = lane >> 3;
  const int cg = (lane & 7) ^ lrow;

  // Of stage s this lane fetches channels 64 s + 8 cg ..: past the last
  // channel (the second half of an odd last stage) both operands are zeros.
  auto past = [&](int s) { return (s * 64 + cg * 8 < cin) ? 0u : 0x80000000u; };
  unsigned b_off[BPW];
  auto issue_b = [&](int slot, int s) {
    unsigned char* sbase_l = smem + slot * SLOT;
    const unsigned bad = past(s);
#pragma unroll
    for (int k = 0; k < BPW; ++k)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsb, (lds_ptr_t)(sbase_l + (BM + 8 * (k * NWAVE + wave)) * ROWB), 16,
          static_cast<int>((b_off[k] + s * ROWB) | bad), 0, 0, 0);
  };
  // The weight rows depend only on the channel block: the first stage's are
  // issued while the tile table is still on its way.
  auto early = [&](int nb) {
#pragma unroll
    for (int k = 0; k < BPW; ++k) {
      const int co = nb * BN + 8 * (k * NWAVE + wave) + lrow;
      b_off[k] = co < cout ? static_cast<unsigned>((co * cin + cg * 8) * 2) : 0x80000000u;
    }
    issue_b(0, 0);
  };
  KTile tl;
  const BlockPos bp = decode_block(a, &tl, early);
  MAFAT_RTRACE(1 + (tl.ch < -1 ? 1 : 0));
  const int wm = wave / WGN, wn = wave - wm * WGN;
  const int M = tl.ch * tl.cw;
  const int m0 = bp.mb * BM, n0 = bp.nb * BN;
  const int sw = tl.sw;
  const int64_t sbase = bp.frame * a.src_fstride + tl.src_off;
  uint16_t* dst = static_cast<uint16_t*>(a.dst) + bp.frame * a.dst_fstride + tl.dst_off;
  const __amdgpu_buffer_rsrc_t rsa = make_rsrc(static_cast<const uint16_t*>(a.src) + sbase,
                                               static_cast<unsigned>((a.src_fstride - tl.src_off) * 2));

  // Scale and bias of this lane's output channels (issued first, so their
  // latency overlaps the main loop).
  float sc[NT][4], bi[NT][4];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    if (POOL) {
      const int co = n0 + wn * WN + j * 16 + (lane & 15);
      const int cc = co < cout ? co : 0;
      sc[j][0] = a.scale[cc];
      bi[j][0] = a.bias[cc];
    } else {
      const int co = n0 + wn * WN + j * 16 + 4 * (lane >> 4);
      const int cc = co < cout ? co : 0;
      const f32x4 s4 = *reinterpret_cast<const f32x4*>(a.scale + cc);
      const f32x4 b4 = *reinterpret_cast<const f32x4*>(a.bias + cc);
#pragma unroll
      for (int r = 0; r < 4; ++r) { sc[j][r] = s4[r]; bi[j][r] = b4[r]; }
    }
  }

  unsigned a_off[APW];
#pragma unroll
  for (int k = 0; k < APW; ++k) {
    const int m = m0 + 8 * (k * NWAVE + wave) + lrow;
    int oy, ox;
    row_pixel<POOL>(tl, m < M ? m : 0, &oy, &ox);
    const int off = (((oy - tl.sy0) * sw + (ox - tl.sx0)) * cin + cg * 8) * 2;
    a_off[k] = (m < M) ? static_cast<unsigned>(off) : 0x80000000u;
  }

  // Stage s's loads (the first stage's weights were issued during the decode).
  auto issue = [&](int slot, int s) {
    unsigned char* sbase_l = smem + slot * SLOT;
    const unsigned bad = past(s);
#pragma unroll
    for (int k = 0; k < APW; ++k)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsa, (lds_ptr_t)(sbase_l + (8 * (k * NWAVE + wave)) * ROWB), 16,
          static_cast<int>((a_off[k] + s * ROWB) | bad), 0, 0, 0);
    if (s != 0) issue_b(slot, s);
  };

  // Fragment reads: lane l supplies rows (l & 15) of a 16-row fragment at K
  // offset 8 (l >> 4) of the 64-byte half h, i.e. global chunk 4h + (l >> 4)
  // of the row, stored at position chunk ^ (row & 7) (row & 7 == l & 7).
  int rd_a[NH], rd_b[NH];
#pragma unroll
  for (int hi = 0; hi < NH; ++hi) {
    const int cpos = (((hi * 4) + (lane >> 4)) ^ (lane & 7)) * 16;
    rd_a[hi] = (wm * WM + (lane & 15)) * ROWB + cpos;
    rd_b[hi] = (BM + wn * WN + (lane & 15)) * ROWB + cpos;
  }

  f32x4 acc[NT][MT];  // [channel tile][pixel tile]
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int slot) {
    const unsigned char* sp = smem + slot * SLOT;
    u32x4 af[NH][MT], bfr[NH][NT];
#pragma unroll
    for (int hi = 0; hi < NH; ++hi) {
#pragma unroll
      for (int i = 0; i < MT; ++i) af[hi][i] = *reinterpret_cast<const u32x4*>(sp + rd_a[hi] + i * 16 * ROWB);
#pragma unroll
      for (int j = 0; j < NT; ++j) bfr[hi][j] = *reinterpret_cast<const u32x4*>(sp + rd_b[hi] + j * 16 * ROWB);
    }
#pragma unroll
    for (int hi = 0; hi < NH; ++hi)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          if constexpr (POOL) mma<MAFAT_BF16>(acc[j][i], af[hi][i], bfr[hi][j]);
          else mma<MAFAT_BF16>(acc[j][i], bfr[hi][j], af[hi][i]);
        }
  };

  // Prologue: stages 0 .. NS-2 in flight.
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < nstage) issue(p, p);
  int slot = 0;
  for (int s = 0; s < nstage; ++s) {
    wait_stage<LPS, NS - 2>(nstage - 1 - s);
    wg_barrier();
    MAFAT_RTRACE(8 + s);
    if (s + NS - 1 < nstage) issue(slot == 0 ? NS - 1 : slot - 1, s + NS - 1);
    compute(slot);
    slot = (slot == NS - 1) ? 0 : slot + 1;
  }

  MAFAT_RTRACE(4);
  // Epilogue: folded batch-norm, activation (leaky: max(v, 0.1 v)), the
  // fused pool, round to bf16; the block's outputs are staged in LDS as rows
  // of BN channels per output pixel and leave as 16-byte stores (each
  // pixel's BN channels one contiguous run); only the tile's own output
  // rectangle is stored.
  constexpr int NTHR = 64 * NWAVE;
  constexpr int RSB = BN * 2 + 16;          // LDS bytes per staged pixel row
  constexpr int NPXO = POOL ? BM / 4 : BM;  // output pixels of the block
  constexpr int CPB = BN / 8;               // 16-byte chunks per pixel row
  static_assert(NPXO * RSB <= NS * SLOT, "staged block fits in the ring");
  const float slope = act_slope(a.act);
  __syncthreads();  // every wave is done with the ring
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if (POOL) {
        const int rl = wm * WM + i * 16 + 4 * (lane >> 4);  // first block row of this lane's window
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(acc[j][i][r], sc[j][0], bi[j][0]);
        float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
        mx = fmaxf(mx, slope * mx);
        store1(reinterpret_cast<uint16_t*>(smem + (rl >> 2) * RSB) + wn * WN + j * 16 + (lane & 15), mx);
      } else {
        const int rl = wm * WM + i * 16 + (lane & 15);
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = fmaf(acc[j][i][r], sc[j][r], bi[j][r]);
          v[r] = fmaxf(v[r], slope * v[r]);
        }
        store4<MAFAT_BF16>(reinterpret_cast<uint16_t*>(smem + rl * RSB) + wn * WN + j * 16 + 4 * (lane >> 4), v);
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < NPXO * CPB; e += NTHR) {
    const int p = e / CPB, k = e - p * CPB;
    const int m = m0 + (POOL ? 4 * p : p);
    const int c0 = n0 + k * 8;
    if (m < M && c0 < cout) {
      int oy, ox;
      if (POOL) {
        const int pw = tl.cw >> 1, qq = m >> 2, qy = qq / pw;
        oy = (tl.cy0 >> 1) + qy;
        ox = (tl.cx0 >> 1) + (qq - qy * pw);
      } else {
        row_pixel<false>(tl, m, &oy, &ox);
      }
      const u32x4 v = *reinterpret_cast<const u32x4*>(smem + p * RSB + k * 16);
      *reinterpret_cast<u32x4*>(dst + ((oy - tl.dy0) * tl.dw + (ox - tl.dx0)) * cout + c0) = v;
    }
  }
  MAFAT_RTRACE(5);
  MAFAT_WG_MARK(g_wg_ring, 1);
}

template <bool POOL>
hipError_t launch_ring_p(const MfmaShape& sh, const StageArgs& args, hipStream_t stream, LaunchEvents ev) {
  const dim3 grid(static_cast<unsigned>(args.total_blocks), args.copy_blocks > 0 ? 2u : 1u);
#define MAFAT_RING(bm_, bn_, wgm_, wgn_, ns_)                                                       \
  if (sh.bm == (bm_) && sh.bn == (bn_) && sh.wgm == (wgm_) && sh.wgn == (wgn_) && sh.depth == (ns_)) { \
    hipExtLaunchKernelGGL((conv_ring_kernel<bm_, bn_, wgm_, wgn_, ns_, POOL>), grid,               \
                          dim3(64 * (wgm_) * (wgn_)), 0, stream, ev.start, ev.stop, 0, args);      \
    return hipGetLastError();                                                                      \
  }
  MAFAT_RING_SHAPES
  MAFAT_RING_TUNE_SHAPES
#undef MAFAT_RING
  return hipErrorInvalidValue;
}

}  // namespace

#ifdef MAFAT_TUNING
extern "C" int mafat_debug_wg_ring(long long* host_out) {
  return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(g_wg_ring), sizeof(g_wg_ring)) == hipSuccess ? 0 : -1;
}
extern "C" int mafat_debug_ring_trace(long long* host_out) {
  return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(g_ring_trace), sizeof(g_ring_trace)) == hipSuccess ? 0 : -1;
}
#endif

hipError_t launch_conv_ring(bool pool, const MfmaShape& shape, const StageArgs& args,
                            hipStream_t stream, LaunchEvents ev) {
  if (args.total_blocks <= 0) return hipSuccess;
  return pool ? launch_ring_p<true>(shape, args, stream, ev) : launch_ring_p<false>(shape, args, stream, ev);
}

}  // namespace mafat
