// The workspace of the MLP calls, and the arithmetic of the hand-over state that the single-launch form keeps in it.
// Plain C++ without HIP: the kernels, the host code and the test that plays calls through on the CPU share it.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace blast_dev {

// ---- control block -------------------------------------------------------------------------------------------------
// In 64-bit words:  [0] signature   [kCtlStatusWord] status (low 32 bits)   [ctl_mark(i)] marks, one at the start of every
// further 512 bytes and one at the very end   [ctl_counter(g)] arrival counter of group g, each in a 128-byte line of its
// own, never at its start.
//
// The block sets itself up: it is whole when the signature is one and every mark fits it.  A signature is never given
// twice (the time of the set-up is in it), so that a block which something else has been written over - memory that an
// allocator hands round, a workspace that begins elsewhere in the same memory - is found out, unless what was written lies
// within 512 bytes and leaves their first word alone.
constexpr int kCtlGroups = 64;
constexpr int kCtlLineWords = 16;
constexpr int kCtlMarkWords = 64;
constexpr int kCtlWords = (2 + kCtlGroups) * kCtlLineWords;
constexpr int kCtlMarks = kCtlWords / kCtlMarkWords + 1;
constexpr int kCtlBytes = kCtlWords * 8;
static_assert(kCtlWords % kCtlMarkWords != 0 && (kCtlWords - 1) % kCtlMarkWords != 0, "the last piece is a part of one");
constexpr int kCtlStatusWord = 2;
constexpr int ctl_counter(int group) { return (2 + group) * kCtlLineWords + 8; }
constexpr int ctl_mark(int i) { return i + 1 < kCtlMarks ? (i + 1) * kCtlMarkWords : kCtlWords - 1; }

constexpr int kCtlEpochBits = 44;
constexpr uint64_t kCtlEpochMask = (uint64_t(1) << kCtlEpochBits) - 1;
constexpr uint64_t kCtlMagic = 0xB1A57;                  // top 20 bits of a signature
constexpr uint64_t kCtlBusy = 0xB1A58B0057EED00Dull;     // in the place of a signature: a wave is setting the block up
static_assert(kCtlMagic >> (64 - kCtlEpochBits) == 0 && kCtlBusy >> kCtlEpochBits != kCtlMagic, "a signature is never busy");
// `clock`: a counter of 100 MHz.  A launch takes longer than one of the ticks of 640 ns that a signature counts, so that the
// epoch, which begins at the time of the set-up and advances by one per launch, stays behind the clock: no epoch comes back
// when the block is set up again, and a word or slot that was left by another launch of a recorded call never fits.
constexpr uint64_t ctl_signature(uint64_t clock) { return (kCtlMagic << kCtlEpochBits) | ((clock >> 6) & kCtlEpochMask); }
constexpr bool ctl_is_signature(uint64_t word) { return word >> kCtlEpochBits == kCtlMagic; }
// (time in the low bits, position in the top ones: fits neither another mark nor another set-up's)
constexpr uint64_t ctl_mark_value(uint64_t signature, int i) { return signature ^ (uint64_t(i + 1) << kCtlEpochBits); }

// A launch adds exactly 2^kCtlShift to every counter, whatever its shape, so that calls of every shape share one control
// block: counter >> kCtlShift, the epoch, is one number for all workgroups of a launch and another in the next launch.
// Workgroup n belongs to group n % kCtlGroups; it adds 1 when it leaves, the first workgroup of a group the rest up to
// 2^kCtlShift as well.
constexpr int kCtlShift = 64 - kCtlEpochBits;
constexpr int64_t kCtlMaxWorkgroups = (int64_t)kCtlGroups << kCtlShift;  // of a launch: 2^20 in a group
constexpr int ctl_group(int workgroup) { return workgroup % kCtlGroups; }
constexpr uint64_t ctl_arrival(int workgroup, int workgroups) {
  if (workgroup >= kCtlGroups) return 1;
  const int members = workgroups / kCtlGroups + (workgroup < workgroups % kCtlGroups ? 1 : 0);
  return (uint64_t(1) << kCtlShift) - uint64_t(members) + 1;
}
// Groups without a member, [n, kCtlGroups) of a launch of n < kCtlGroups workgroups: workgroup 0 adds for them.
constexpr uint64_t kCtlArrivalOfNone = uint64_t(1) << kCtlShift;
constexpr uint64_t ctl_epoch(uint64_t counter) { return counter >> kCtlShift; }
// Whether a counter can be one of the block with this signature (of any age that occurs), not what stood there before.
constexpr bool ctl_epoch_fits(uint64_t epoch, uint64_t signature) { return ((epoch - signature) & kCtlEpochMask) >> 32 == 0; }
// What the set-up writes into word `i` > 0 of the block.
constexpr uint64_t ctl_initial(int i, uint64_t signature) {
  if (i % kCtlMarkWords == 0) return ctl_mark_value(signature, i / kCtlMarkWords - 1);
  if (i == kCtlWords - 1) return ctl_mark_value(signature, kCtlMarks - 1);
  return i % kCtlLineWords == 8 ? signature << kCtlShift : 0;  // (the counters, and two words that nobody reads)
}

// ---- workspace -----------------------------------------------------------------------------------------------------
// The control block lies at byte 0 for every shape, token count and path, and everything a call writes lies behind it:
// what one call leaves there is whole when the next call of whatever shape finds it.
constexpr size_t ws_align(size_t x) { return (x + 255) / 256 * 256; }
constexpr size_t mlp_h_bytes(int64_t I, int64_t T) { return ws_align((size_t)T * (size_t)I * 2); }
constexpr size_t mlp_slot_bytes(int64_t I) { return ws_align((size_t)(I / 16) * 8); }
constexpr size_t kMlpCtlOffset = 0;
constexpr size_t kMlpHOffset = kCtlBytes;  // H in bf16, token-major [T][I] (whole lines: see the consumers' reads)
constexpr size_t mlp_slot_offset(int64_t I, int64_t T) { return kMlpHOffset + mlp_h_bytes(I, T); }  // a 64-bit word per 16 rows of H
constexpr size_t mlp_workspace_bytes(int64_t I, int64_t T) { return mlp_slot_offset(I, T) + mlp_slot_bytes(I); }
static_assert(kMlpHOffset % 256 == 0, "H starts on a line");
// H as tagged words, behind that where the caller's workspace has room.
constexpr int kTaggedTokens = 4;
constexpr size_t tagged_offset(int64_t I, int64_t T) { return mlp_workspace_bytes(I, T); }
constexpr size_t tagged_bytes(int32_t b, int64_t I, int64_t T) {
  return (b == 64 || b == 128) && T <= kTaggedTokens ? (size_t)T * (size_t)I * 8 : 0;
}
// What the queries ask for: enough for every smaller call as well, so that a program that asks once, for its largest batch,
// has the words at the smaller ones.
constexpr size_t mlp_query_bytes(int32_t b, int64_t I, int64_t T) {
  const int64_t few = T < kTaggedTokens ? T : kTaggedTokens;
  const size_t own = mlp_workspace_bytes(I, T), smaller = mlp_workspace_bytes(I, few) + tagged_bytes(b, I, few);
  return own > smaller ? own : smaller;
}

}  // namespace blast_dev
