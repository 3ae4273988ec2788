// Lexical anchoring (Sec. 3.3): longest-suffix n-gram match over the context.
//
// One workgroup per sequence, on 64-bit words of positions.  A wave reads 64
// consecutive tokens with one load (lane = position) and compares them with
// suffix token k = M[L-1-k]: the compare's lane mask is the word of
// E_k = {i : M[i] == M[L-1-k]}, one VALU instruction per 64 positions.  The
// ends of matches of length n or more are
//   B_n = E_0 & (E_1 << 1) & ... & (E_{n-1} << (n-1)),
// where the bits shifted in come from the previous word's tokens (n_max is at
// most 64, so one word back suffices; below position 0 they are zero, so an
// n-gram never starts before the context).  Most words have no bit in E_0 and
// cost one compare; the others extend level by level in scalar registers
// until nothing is left.  Each word keeps its longest level and that level's
// members in LDS; the workgroup's longest level is n*, and the members of the
// words that reached it, prefix-summed, are C_lex in ascending order.
//
// What bounds it: a trip to memory for the length and the tokens (requested
// together; a row that fits the waves' registers also takes its suffix from
// them), and the instructions of the one CU that a sequence gets: every
// instruction, scalar ones included, takes 4 cycles of its SIMD, and code that
// runs once per launch is fetched at about 0.4 us per KiB, so the loops below
// are kept short rather than unrolled for every case.  Back-to-back calls, us
// (in brackets the kernel before: a run of positions per thread over tokens
// staged in LDS, in two passes per 32768-token piece): 4 x 131072 tokens
// 13.8-17.2 (104-128), 8 x 32768 5.8-6.7 (9.3-9.6), 16 x 8192 4.0-4.3
// (4.4-4.7), 1 x 4096 3.1 (3.6), 1 x 512 2.8 (3.4).
#include "adapld_internal.h"
#include "device_utils.h"

namespace adapld {
namespace {

constexpr int kLexThreads = 1024;
constexpr int kLexWaves = kLexThreads / kWave;
constexpr int kLexWords = 8192;        // words per piece (524288 tokens)

// v with lane `l` replaced by the uniform value x (the compiler has no builtin
// for the instruction, so its intrinsic is named).
extern "C" __device__ uint32_t write_lane(uint32_t x, uint32_t l, uint32_t v) __asm("llvm.amdgcn.writelane.i32");

// R: words one wave has in flight (and as many behind them).  ONE: the waves'
// registers hold every row whole (L_stride <= R * kLexThreads), which leaves
// out the loops over batches and pieces and the code that they run once.
template <int R, bool ONE>
__global__ __launch_bounds__(kLexThreads) void lexical_match_kernel(
    const int32_t* __restrict__ tokens, const int32_t* __restrict__ lens, int L_stride, int n_max,
    int32_t* __restrict__ cand_pos, int32_t* __restrict__ cand_count,
    int32_t* __restrict__ match_n) {
  __shared__ uint64_t s_bits[kLexWords];   // members of the word's longest level
  __shared__ uint8_t s_lv[kLexWords];      // that level (0: no match ends in the word)
  __shared__ int s_slot[ONE ? R * kLexWaves : 1];   // first output slot of every word
  __shared__ int s_suffix[kWave];
  __shared__ int s_red[2][kLexWaves];

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int32_t* __restrict__ M = tokens + (size_t)b * L_stride;
  const int row_words = (L_stride + kWave - 1) / kWave;
  const int piece = min(kLexWords, row_words);
  const int per = (piece + kLexWaves - 1) / kLexWaves;   // contiguous words per wave and piece
  const int f0 = wave * per;

  // Words [w, w + R) of the row, one token per lane; positions past the row
  // re-read its last token.
  auto load_words = [&](int w, int (&t)[R]) {
    const int p0 = w * kWave;
    if (p0 + R * kWave <= L_stride) {
#pragma unroll
      for (int i = 0; i < R; ++i) t[i] = (M + p0)[i * kWave + lane];
    } else {
      const int q0 = min(p0, L_stride - 1);
      const int room = L_stride - 1 - q0;
#pragma unroll
      for (int i = 0; i < R; ++i) t[i] = (M + q0)[min(i * kWave + lane, room)];
    }
  };
  auto load_before = [&](int w) { return M[min(max(w - 1, 0) * kWave + lane, L_stride - 1)]; };

  // The first tokens are requested before the length is known.
  int tok[R];
  load_words(f0, tok);
  int before = load_before(f0);   // the word before (unused for word 0)
  const int L = min(max(lens[b], 0), L_stride);
  // Lane k's suffix token: from the tokens in registers when they hold the
  // whole row, else by a load that waits for the length.
  int suf;
  if (ONE || (per <= R && kLexWaves * per >= row_words)) {
    const int p0 = f0 * kWave;
    if (p0 < L && p0 + per * kWave > L - n_max) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int k = L - 1 - (p0 + i * kWave + lane);
        if (i < per && k >= 0 && k < n_max) s_suffix[k] = tok[i];
      }
    }
    __syncthreads();
    suf = s_suffix[lane];
  } else {
    suf = M[max(L - 1 - lane, 0)];
  }

  const int J = max(L - 1, 0);                     // candidate ends are [0, J)
  const int words = (J + kWave - 1) / kWave;
  const int npieces = ONE ? 1 : (words + piece - 1) / piece;
  int32_t* __restrict__ out = cand_pos + (size_t)b * L_stride;
  const int s0 = __builtin_amdgcn_readlane(suf, 0);

  // Fills s_bits and s_lv for the piece's words [w0, w0 + n) (the last batch's
  // also stay in lanes 1 .. R); returns the longest level of this lane's words.
  uint64_t bits = 0ull;
  int lv = 0;
  auto fill = [&](int w0, int n, bool loaded) {
    int best = 0;
    const int w_end = min(per, n - f0);            // this wave's words (may be <= 0)
    const int end = min((w0 + f0 + w_end) * kWave, J);   // its candidate ends stop here
    if (!ONE && !loaded && w_end > 0) {
      load_words(w0 + f0, tok);
      before = load_before(w0 + f0);
    }
    for (int i0 = 0; i0 < w_end; i0 += R) {
      const int f = f0 + i0;
      const int p0 = (w0 + f) * kWave;
      int nxt[R];
      if (!ONE && i0 + R < w_end) load_words(w0 + f + R, nxt);
      // A token that is no candidate end of this wave must not match (nor is
      // it read as the token before one).
      if (p0 + R * kWave > end) {
#pragma unroll
        for (int i = 0; i < R; ++i) tok[i] = i * kWave + lane < end - p0 ? tok[i] : ~s0;
      }
      // Lane 1 + i holds word i of every level's set, lane 0 the word before
      // the batch, so one pass of vector arithmetic extends all R words.
      bits = 0ull;
      lv = 0;
      for (int k = 0;; ++k) {
        const int sk = __builtin_amdgcn_readlane(suf, k);
        uint64_t m = __ballot(before == sk);
        if (p0 == 0) m = 0ull;                     // no token before the row
        uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
#pragma unroll
        for (int i = 0; i < R; ++i) {
          m = __ballot(tok[i] == sk);
          lo = write_lane((uint32_t)m, 1 + i, lo);
          hi = write_lane((uint32_t)(m >> 32), 1 + i, hi);
        }
        const uint64_t e = ((uint64_t)hi << 32) | lo;
        uint64_t nb;
        if (k == 0) {
          nb = lane >= 1 && lane <= R ? e : 0ull;
        } else {
          // the word before each: the lane below's (wave_shr:1)
          const uint32_t plo = __builtin_amdgcn_mov_dpp(lo, 0x138, 0xf, 0xf, false);
          const uint32_t phi = __builtin_amdgcn_mov_dpp(hi, 0x138, 0xf, 0xf, false);
          nb = lv == k ? bits & ((e << k) | ((((uint64_t)phi << 32) | plo) >> (kWave - k))) : 0ull;
        }
        if (nb) {
          bits = nb;
          lv = k + 1;
        }
        if (k + 1 == n_max || !__ballot(nb != 0ull)) break;
      }
      best = max(best, lv);
      if (lane >= 1 && lane <= min(R, w_end - i0)) {
        s_bits[f + lane - 1] = bits;
        s_lv[f + lane - 1] = (uint8_t)lv;
      }
      if (ONE) break;
      before = tok[R - 1];
#pragma unroll
      for (int i = 0; i < R; ++i) tok[i] = nxt[i];
    }
    return best;
  };

  // One piece is filled once, reduced to n* and compacted from LDS; several
  // are filled in order for n*, then each again for its members.
  int best = 0, n_star = 0, total = 0;
  const int rounds = npieces > 1 ? 2 * npieces : npieces;
  for (int q = 0; q < rounds; ++q) {
    const int p = q < npieces ? q : q - npieces;
    const int w0 = p * piece;
    const int n = min(piece, words - w0);
    best = max(best, fill(w0, n, q == 0));
    if (q == npieces - 1) {
      best = wave_max_i32(best);
      if (lane == 0) s_red[0][wave] = best;
      __syncthreads();
      n_star = wave_max_i32(s_red[0][lane & (kLexWaves - 1)]);
      if (n_star == 0) break;
      if (npieces > 1) continue;
    } else if (n_star == 0) {
      continue;
    }
    // Each thread takes one word per round (neighbouring lanes neighbouring
    // words, so the slots of a round follow thread order).
    for (int i0 = 0; i0 < n; i0 += kLexThreads) {
      if (!ONE && (npieces > 1 || i0 > 0)) __syncthreads();   // the words are filled; earlier reads of s_red[1] are done
      const int i = i0 + tid;
      uint64_t v = i < n && s_lv[i] == n_star ? s_bits[i] : 0ull;
      const int cnt = __popcll(v);
      const int incl = wave_incl_scan_i32(cnt);
      if (lane == kWave - 1) s_red[1][wave] = incl;
      __syncthreads();
      const int sums = wave_incl_scan_i32(lane < kLexWaves ? s_red[1][lane & (kLexWaves - 1)] : 0);
      int slot = total + incl - cnt + (wave > 0 ? __builtin_amdgcn_readlane(sums, wave - 1) : 0);
      total += __builtin_amdgcn_readlane(sums, kWave - 1);
      // A context of few tokens (more than 8 members per word): every wave writes
      // its own words, one lane per member, instead of one lane all members of a
      // word.  us a call, tokens all equal: 512 5.3 -> 3.0, 64 x 2048 5.8 -> 3.6,
      // 16 x 8192 7.5 -> 5.0.  Where words have a few members, one lane each is
      // the shorter way: 16 x 8192 Zipf tokens 4.1, word by word 4.9.
      if (ONE && total > 8 * n) {
        if (i < n) s_slot[i] = slot;
        __syncthreads();
        for (int e = 1; e <= min(R, n - f0); ++e) {
          const uint64_t word = __builtin_amdgcn_readlane(lv, e) == n_star ? readlane_u64(bits, e) : 0ull;
          const int before_lane = __builtin_amdgcn_mbcnt_hi((uint32_t)(word >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)word, 0u));
          if ((word >> lane) & 1ull) out[s_slot[f0 + e - 1] + before_lane] = (f0 + e - 1) * kWave + lane;
        }
        break;
      }
      while (v) {
        const int e = __builtin_ctzll(v);
        v &= v - 1;
        out[slot++] = (w0 + i) * kWave + e;
      }
      if (ONE) break;                      // at most 128 words
    }
    if (npieces > 1) __syncthreads();     // the piece has been read before the next fill
  }
  if (tid == 0) {
    cand_count[b] = total;
    match_n[b] = n_star;
  }
}

}  // namespace

hipError_t launch_lexical_match(const int32_t* tokens, const int32_t* lens, int B, int L_stride,
                                int n_max, int32_t* cand_pos, int32_t* cand_count,
                                int32_t* match_n, hipStream_t stream) {
  // The least R whose 16 waves hold a row of the batch whole in one pass: less
  // code and fewer compares of empty words (1 x 4096 tokens 3.1 us with 4
  // words per wave, 4.0 with 8 and the loops; 1 x 512 2.8 against 3.1).
  // Longer rows loop over batches of 16 words.
  auto kernel = L_stride <= 1 * kLexThreads   ? lexical_match_kernel<1, true>
                : L_stride <= 2 * kLexThreads ? lexical_match_kernel<2, true>
                : L_stride <= 4 * kLexThreads ? lexical_match_kernel<4, true>
                : L_stride <= 8 * kLexThreads ? lexical_match_kernel<8, true>
                                              : lexical_match_kernel<16, false>;
  hipLaunchKernelGGL(kernel, dim3(B), dim3(kLexThreads), 0, stream, tokens, lens,
                     L_stride, n_max, cand_pos, cand_count, match_n);
  return hipGetLastError();
}

}  // namespace adapld
