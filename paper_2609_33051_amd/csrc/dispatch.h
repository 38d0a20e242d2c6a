// Maps a runtime shape to its compiled kernel instantiation and launches it.
// Compiled shapes: (K, V) in {(64,64), (128,64), (128,128)}; R in {8, 16, 32, K}
// (update also R = 0); windows up to 16 or 32 slots; fp32 or bf16 io; fp32 or
// bf16 sketch.
#pragma once

#include <hip/hip_runtime.h>

#include "decode.h"
#include "update.h"

namespace skssm {

constexpr int kUnsupported = -2;

// LDS of one gfx950 CU, shared by the workgroups resident on it.
constexpr size_t kLdsPerCU = 160 * 1024;

// Dynamic LDS (unused by the kernel) that holds a kernel to at most `cap`
// resident workgroups per CU: each then takes more than a (cap + 1)-th of the
// CU's LDS.  Zero where the kernel's static LDS already does that, or if its
// attributes cannot be read (the launch then runs uncapped).
template <typename Kernel>
size_t lds_for_cap(Kernel kern, int cap) {
  hipFuncAttributes at;
  if (hipFuncGetAttributes(&at, reinterpret_cast<const void*>(kern)) != hipSuccess) return 0;
  const size_t need = kLdsPerCU / (size_t)(cap + 1) + 1024;
  return need > at.sharedSizeBytes ? need - at.sharedSizeBytes : 0;
}

// Resident workgroups per CU for the kernels that read each item's state and
// write it back in place (the flush with the offline map or none, and the
// single-token update; 0: what registers and LDS allow).  With more of these
// streams in flight per CU the in-place stream runs slower; with too few, each
// workgroup's own latency shows.  The line lies by the bytes of an item's state
// (4 K V) and the work between its load and store, measured at 1 GiB of state
// (us at a cap of two / three / four / five / none):
//   Mamba-2  16 KB  582 / 461 / 429 / 425 / 443     -> 5
//            32 KB  433 / 397 / 422 / 438 / 444     -> 3
//            64 KB  425 / 459 / 465 / 475 / 471     -> 2
//   GDN      16 KB  672 / 559 / 497 / 470 / 450     -> none
//            32 KB  575 / 489 / 440 / - / 436       -> none
//            64 KB  456 / 432 / - / - / 421..452    -> 3  (KDA 470 / 446 / - / - / 477)
// (rank 16, W = 16, bf16 inputs).  Wider inputs or a larger rank move it (us at
// the cap above / at the one taken, 1 GiB of state): Mamba-2 16 KB fp32 inputs rank 0 428 / 417,
// rank 16, W = 32 577 / 563; 32 KB rank 32, W = 16, bf16 437 / 418; 64 KB rank
// 32, W = 32, bf16 478 / 441.
// The flushes that build a state-dependent map and the decode do arithmetic or
// wait on latency between their loads and keep their occupancy (capping them
// measured slower), as does the initial sketch (a read of the state, run once
// after prefill); but for Mamba-2's 32 KB items at rank 8 with fp32 inputs,
// W <= 16: six of those (with 12 KB of inputs each and the least arithmetic) run
// slower than five (us at six / five, 1 GiB of state, fp32 / bf16 sketch: P = 4
// 509, 479 / 495, 470; exact 502, 470 / 485, 465; bf16 inputs P = 4 447, 435 /
// 454, 453; rank 16 exact, fp32 inputs 554, 518 / 562, 553).
template <int KIND, int K, int V, int R, int WM, typename IO, int P>
constexpr int flush_cap() {
  constexpr int kb = 4 * K * V / 1024;
  constexpr bool narrow = sizeof(IO) == 2;
  if (P != 0) return KIND == MAMBA2 && kb == 32 && R == 8 && WM == 16 && !narrow ? 5 : 0;
  if (KIND != MAMBA2) return kb >= 64 ? 3 : 0;
  if (kb >= 64) return R == 32 && WM == 32 && narrow ? 3 : 2;
  if (kb >= 32) return R == 32 && WM == 16 && narrow ? 4 : 3;
  return narrow || R >= 32 ? 5 : R > 0 ? 4 : 3;
}

// Bytes of state in flight per CU of the single-token update, whose workgroups
// are one 16-value tile each (us at four / five / six / eight tiles of 8 KB and
// uncapped, 1 GiB of state: GDN K = V = 128 332 / 322 / 329 / 346 / 353, Mamba-2
// K = 128, V = 64 332 / 340 / 345 / 360 / 348; at eight / ten / twelve tiles of
// 4 KB and uncapped: GDN K = V = 64 334 / 329 / 333 / 346, Mamba-2 329 / 334 /
// 332 / 348).  The erase families wait for the tile's product with k before
// their first store and take a little more.
constexpr int token_bytes_per_cu(int kind) { return (kind == MAMBA2 ? 32 : 40) * 1024; }

template <int KIND, int K, int V, int R, int WM, typename IO, typename SK, int P, bool APPEND>
int launch_decode_as(const DecodeArgs& a, hipStream_t s) {
  const unsigned tiles = (unsigned)((a.B + 3) / 4);
  if (a.ndense > 0)
    hipLaunchKernelGGL((decode_kernel<KIND, K, V, R, WM, IO, SK, P, true, APPEND>), dim3((unsigned)a.H * tiles), dim3(256), 0,
                       s, a);
  else
    hipLaunchKernelGGL((decode_kernel<KIND, K, V, R, WM, IO, SK, P, false, APPEND>), dim3((unsigned)a.H * tiles), dim3(256), 0,
                       s, a);
  return 0;
}

template <int KIND, int K, int V, int R, int WM, typename IO, typename SK, int P>
int launch_decode(const DecodeArgs& a, hipStream_t s) {
  return a.append ? launch_decode_as<KIND, K, V, R, WM, IO, SK, P, true>(a, s)
                  : launch_decode_as<KIND, K, V, R, WM, IO, SK, P, false>(a, s);
}

template <int KIND, int K, int V, int WM, typename IO>
int launch_full_read(const DecodeArgs& a, hipStream_t s) {
  const unsigned groups = (unsigned)(((size_t)a.B * a.H + 3) / 4);
  if (a.append)
    hipLaunchKernelGGL((full_read_kernel<KIND, K, V, WM, IO, true>), dim3(groups), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((full_read_kernel<KIND, K, V, WM, IO, false>), dim3(groups), dim3(256), 0, s, a);
  return 0;
}

template <int KIND, int K, int V, int R, int WM, typename IO, typename SK, int P>
int launch_update(const UpdateArgs& a, hipStream_t s) {
  const size_t items = (size_t)a.B * a.H;
  constexpr int kCap = flush_cap<KIND, K, V, R, WM, IO, P>();
  static const size_t cap = kCap ? lds_for_cap(&update_kernel<KIND, K, V, R, WM, IO, SK, P>, kCap) : 0;
  hipLaunchKernelGGL((update_kernel<KIND, K, V, R, WM, IO, SK, P>), dim3((unsigned)items), dim3(256), a.nt > 0 ? cap : 0,
                     s, a);
  return 0;
}

// State-dependent maps: piv = 4 (P = 4 pivots) is compiled for ranks 8..32,
// piv = -1 (the exact metric, flush only: decode reads either map the same
// way) for ranks 8 and 16.
template <int R> constexpr bool kPivotRank = R >= 8 && R <= 32;
template <int R> constexpr bool kExactRank = R == 8 || R == 16;

template <int KIND, int K, int V, int R, int WM, int P>
int decode_t(const DecodeArgs& a, int io, int sk, hipStream_t s) {
  if (io) return sk ? launch_decode<KIND, K, V, R, WM, bf16_t, bf16_t, P>(a, s) : launch_decode<KIND, K, V, R, WM, bf16_t, float, P>(a, s);
  return sk ? launch_decode<KIND, K, V, R, WM, float, bf16_t, P>(a, s) : launch_decode<KIND, K, V, R, WM, float, float, P>(a, s);
}

template <int KIND, int K, int V, int R>
int decode_w(const DecodeArgs& a, int io, int sk, int piv, hipStream_t s) {
  if constexpr (kPivotRank<R>) {
    if (piv) return a.W <= 16 ? decode_t<KIND, K, V, R, 16, 4>(a, io, sk, s) : decode_t<KIND, K, V, R, 32, 4>(a, io, sk, s);
  } else {
    if (piv) return kUnsupported;
  }
  return a.W <= 16 ? decode_t<KIND, K, V, R, 16, 0>(a, io, sk, s) : decode_t<KIND, K, V, R, 32, 0>(a, io, sk, s);
}

// One (kind, K, V) shape; explicitly instantiated in its own translation unit.
template <int KIND, int K, int V>
int decode_r(const DecodeArgs& a, int R, int io, int sk, int piv, hipStream_t s) {
  switch (R) {
    case 8: return decode_w<KIND, K, V, 8>(a, io, sk, piv, s);
    case 16: return decode_w<KIND, K, V, 16>(a, io, sk, piv, s);
    case 32: return decode_w<KIND, K, V, 32>(a, io, sk, piv, s);
    case K: return decode_w<KIND, K, V, K>(a, io, sk, piv, s);
    default: return kUnsupported;
  }
}

template <int KIND>
int run_decode(const DecodeArgs& a, int K, int V, int R, int io, int sk, int piv, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (K == 64 && V == 64) return decode_r<KIND, 64, 64>(a, R, io, sk, piv, s);
  if (K == 128 && V == 64) return decode_r<KIND, 128, 64>(a, R, io, sk, piv, s);
  if (K == 128 && V == 128) return decode_r<KIND, 128, 128>(a, R, io, sk, piv, s);
  return kUnsupported;
}

template <int KIND, int K, int V>
int full_read_w(const DecodeArgs& a, int io, hipStream_t s) {
  if (a.W <= 16)
    return io ? launch_full_read<KIND, K, V, 16, bf16_t>(a, s) : launch_full_read<KIND, K, V, 16, float>(a, s);
  return io ? launch_full_read<KIND, K, V, 32, bf16_t>(a, s) : launch_full_read<KIND, K, V, 32, float>(a, s);
}

template <int KIND>
int run_full_read(const DecodeArgs& a, int K, int V, int io, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (K == 64 && V == 64) return full_read_w<KIND, 64, 64>(a, io, s);
  if (K == 128 && V == 64) return full_read_w<KIND, 128, 64>(a, io, s);
  if (K == 128 && V == 128) return full_read_w<KIND, 128, 128>(a, io, s);
  return kUnsupported;
}

template <int KIND, int K, int V, typename IO>
int launch_token(const UpdateArgs& a, hipStream_t s) {
  const size_t tiles = (size_t)a.B * a.H * (V / 16);  // < 2^26 (the ABI bounds B*H)
  static const size_t cap = lds_for_cap(&token_kernel<KIND, K, V, IO>, token_bytes_per_cu(KIND) / (64 * K));
  hipLaunchKernelGGL((token_kernel<KIND, K, V, IO>), dim3((unsigned)tiles), dim3(64), cap, s, a);
  return 0;
}

// Whether a single token's update may run as token_kernel: its workgroups, one
// per 16-value tile, each read the item's whole k, q and (KDA) decays, its
// gates and their own values, and write their own part of o in no order among
// themselves.  Where o takes the place of one of those arrays the window's
// kernel runs, one workgroup per item, which has staged them before it writes.
template <int KIND, int K, int V>
bool tiles_independent(const UpdateArgs& a, int io) {
  const size_t items = (size_t)a.B * a.H, slots = a.tk ? items : items * (size_t)a.W, e = io ? 2 : 4;
  const void* in[] = {a.q, a.tk ? a.tk : a.rk, a.tk ? a.tv : a.rv, a.tk ? a.tbeta : a.rbeta, a.tk ? a.tla : a.rla};
  const size_t bytes[] = {items * K * e, slots * K * e, slots * V * e, slots * 4, slots * (KIND == KDA ? K : 1) * 4};
  for (int f = 0; f < 5; ++f)
    if (overlap(a.o, items * V * 4, in[f], bytes[f])) return false;
  return true;
}

template <int KIND, int K, int V, int R, int WM, int P>
int update_t(const UpdateArgs& a, int io, int sk, hipStream_t s) {
  if constexpr (R == 0) {  // no sketch: its dtype does not matter
    // a single token (window-1 decoding, or a window flushed after its first
    // token): the rank-1 update streams the state through registers
    if (a.nt == 1 && tiles_independent<KIND, K, V>(a, io)) return io ? launch_token<KIND, K, V, bf16_t>(a, s) : launch_token<KIND, K, V, float>(a, s);
    return io ? launch_update<KIND, K, V, 0, WM, bf16_t, float, 0>(a, s) : launch_update<KIND, K, V, 0, WM, float, float, 0>(a, s);
  } else {
    if (io) return sk ? launch_update<KIND, K, V, R, WM, bf16_t, bf16_t, P>(a, s) : launch_update<KIND, K, V, R, WM, bf16_t, float, P>(a, s);
    return sk ? launch_update<KIND, K, V, R, WM, float, bf16_t, P>(a, s) : launch_update<KIND, K, V, R, WM, float, float, P>(a, s);
  }
}

template <int KIND, int K, int V, int R>
int update_w(const UpdateArgs& a, int io, int sk, int piv, hipStream_t s) {
  if constexpr (kExactRank<R>) {
    if (piv < 0) return a.W <= 16 ? update_t<KIND, K, V, R, 16, -1>(a, io, sk, s) : update_t<KIND, K, V, R, 32, -1>(a, io, sk, s);
  }
  if constexpr (kPivotRank<R>) {
    if (piv > 0) return a.W <= 16 ? update_t<KIND, K, V, R, 16, 4>(a, io, sk, s) : update_t<KIND, K, V, R, 32, 4>(a, io, sk, s);
  }
  if (piv) return kUnsupported;
  return a.W <= 16 ? update_t<KIND, K, V, R, 16, 0>(a, io, sk, s) : update_t<KIND, K, V, R, 32, 0>(a, io, sk, s);
}

// One (kind, K, V) shape; explicitly instantiated in its own translation unit.
template <int KIND, int K, int V>
int update_r(const UpdateArgs& a, int R, int io, int sk, int piv, hipStream_t s) {
  switch (R) {
    case 0: return update_w<KIND, K, V, 0>(a, io, sk, piv, s);
    case 8: return update_w<KIND, K, V, 8>(a, io, sk, piv, s);
    case 16: return update_w<KIND, K, V, 16>(a, io, sk, piv, s);
    case 32: return update_w<KIND, K, V, 32>(a, io, sk, piv, s);
    case K: return update_w<KIND, K, V, K>(a, io, sk, piv, s);
    default: return kUnsupported;
  }
}

template <int KIND>
int run_update(const UpdateArgs& a, int K, int V, int R, int io, int sk, int piv, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (K == 64 && V == 64) return update_r<KIND, 64, 64>(a, R, io, sk, piv, s);
  if (K == 128 && V == 64) return update_r<KIND, 128, 64>(a, R, io, sk, piv, s);
  if (K == 128 && V == 128) return update_r<KIND, 128, 128>(a, R, io, sk, piv, s);
  return kUnsupported;
}

}  // namespace skssm
