// Small host-side helpers that linfusion.hip shares with the library's other translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lfh {

// LINFUSION_OK when the current device is a gfx950, else LINFUSION_ERR_DEVICE (cached per device)
int check_device();
// `dflt`, unless tuning is switched on (LINFUSION_TUNE=1 at first use, or linfusion_set_tuning) and the
// environment holds a positive integer under `name`
int env_int(const char* name, int dflt);
// compute units of the current device (256 while no device is visible)
int num_cu();

// Element strides {batch, head, token} of a [B, H, N, d] view with contiguous channels (null = dense).
// check_strides: LINFUSION_OK when the kernels can address the view (non-negative, token rows 16-byte aligned,
// index widths); `written` additionally requires that no two rows share memory.  span_bytes: bytes from the
// first to one past the last element the view touches.
int check_strides(const long long s[3], int B, int H, long long N, int d, size_t esz, bool written);
size_t span_bytes(const long long s[3], int B, int H, long long N, int d, size_t esz);

// How a head's tiles are dealt to workgroups of `waves` waves, each of which takes a tile per round: `most` workgroups at
// most, as few as keep the longest at the number of rounds that `most` of them need (every workgroup leaves a partial state
// or stages one), and blocks of up to `blk` consecutive tiles, halved until the longest workgroup's whole blocks are within
// a thirty-second of that number (blocks of 16 tiles, 512 tiles, 25 workgroups: 8 rounds where 6 do).
// us per call, blocks of 16 or 8 tiles whatever the number -> these: bf16 2 x 10 x 16384 x 64 54.0 -> 48.0, fp16 8 x 100000 x
// 40 60.1 -> 55.8, 20 x 65536 x 64 130.2 -> 124.2, fp32 forward and backward 12 x 8 x 4096 x 40 192.4 -> 183.1; fewest
// workgroups: fp16 2 x 5 x 9216 x 64 24.0 -> 23.2, fp32 2 x 10 x 16384 x 64 83.9 -> 82.7.
// `row_bytes`: of a head's rows (of a group of heads: its pieces of a row).  Where they are no whole 128-byte lines,
// neighbouring heads of a token-major tensor share lines.  Workgroups are dealt to the eight XCDs in turn; with 1, 2, 4 or a
// multiple of eight workgroups per head, where the same rounds allow it, the workgroups that walk the same tokens of all,
// every fourth or every second head share an XCD and its L2 (forward and backward of fp16 2 x 10 x 13056 x 16 token-major: 24
// workgroups 73 us, 21 80 us; of bf16 12 x 10 x 1094 x 8: 4 workgroups 41.5 us, 3 45.5 us).  Where eight are too many, rows of
// up to 48 bytes take a multiple of four, with which every second head shares (forward token-major, bf16: 4 x 10 x 9626 x 16
// 10 workgroups 32.3 us, 12 28.2; 2 x 12 x 9443 x 8 22.2, 17.8; 1 x 5 x 135255 x 16 56.9, 48.5; wider rows 0.97 to 1.07,
// contiguous tensors 0.97 to 1.06 either way).
struct Share { int wgs, blk; };   // blk: in tiles, whole rounds
inline Share even_share(long long n_tiles, long long most, int waves, int blk, long long row_bytes = 0) {
  const long long rounds = (n_tiles + waves - 1) / waves;
  long long s = most < rounds ? most : rounds;
  if (s < 1) s = 1;
  const long long longest = (rounds + s - 1) / s;
  const long long room = s;
  s = (rounds + longest - 1) / longest;
  if (row_bytes % 128 != 0) {
    const long long even = s <= 2 ? s : (s <= 4 ? 4 : (s + 7) / 8 * 8), half = (s + 3) / 4 * 4;
    if (even <= room) s = even;
    else if (row_bytes <= 48 && s > 4 && half <= room) s = half;
  }
  long long b = blk / waves;   // rounds per block
  if (b > longest) b = longest;
  if (b < 1) b = 1;
  while (b > 1 && ((rounds + b - 1) / b + s - 1) / s * b * 32 > longest * 33) b /= 2;
  if (b * waves > 1 << 28) b = (1 << 28) / waves;
  return Share{(int)s, (int)(b * waves)};
}

// Whether per-head kernels of that many heads keep nearly all of two workgroups per CU busy with a multiple of eight of them
// per head, so that the heads' workgroups which share cache lines of a token-major tensor share an XCD too.
inline bool heads_fill(long long heads) {
  const long long all = 2 * num_cu(), even = all / heads / 8 * 8;
  return 20 * even * heads >= 17 * all;
}

// true when the byte ranges [a, a + na) and [b, b + nb) share a byte
inline bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

// Workgroups may use up to 160 KiB of LDS on this device; above 64 KiB the kernel has to be told (per kernel; cheap).
template <typename KernelT>
inline bool allow_lds(KernelT kernel, int bytes) {
  if (bytes <= 65536) return true;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) !=
      hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return true;
}

}  // namespace lfh
