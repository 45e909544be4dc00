// Plays sequences of MLP calls through on one workspace, with the layout and the arithmetic of the hand-over that the
// kernels use (csrc/handover.h): no GPU.  The workgroups of a launch look at the control block and leave in a
// random interleaving; every data word that a call writes is written with a value of its own.
//
// stdin: one sequence per line, calls "form:I:E:T[:base]" separated by blanks; the workspace begins `base` bytes into the
// memory (0).  Forms: slots, words (single-launch forms), plain (two launches: H only), low (another use of the memory: 2 T I
// bytes from the base on, as the MLP on E5M2 weights), pieces (another use: 512-byte pieces I to I + T of the memory).
// A call that is written twice stands for a recorded one: it carries the same host token each time, and no two launches of it
// may see the same epoch, whatever happened in between.
// stdout: one line per sequence, "ok" or what went wrong first.
#include <algorithm>
#include <cstdio>
#include <iostream>
#include <random>
#include <set>
#include <sstream>
#include <string>
#include <vector>

#include "../paper_2507_03117_amd/csrc/handover.h"

using namespace blast_dev;

struct Call {
  std::string form;
  int64_t I, E, T, base;
};

static std::string play(const std::vector<Call>& calls, std::mt19937_64& rng) {
  size_t bytes = 0;
  for (const Call& c : calls) bytes = std::max(bytes, c.base + tagged_offset(c.I, c.T) + (size_t)(c.T * c.I * 8));
  std::vector<uint64_t> mem(bytes / 8);
  uint64_t clock = rng() >> 8;
  std::set<std::pair<std::string, uint64_t>> seen;  // (call, epoch)
  for (auto& w : mem) w = rng();
  auto fill = [&](size_t byte, size_t bytes) {
    for (size_t i = byte / 8; i < (byte + bytes + 7) / 8; ++i) mem.at(i) = rng();
  };
  for (size_t n = 0; n < calls.size(); ++n) {
    const Call& c = calls[n];
    auto fail = [&](const char* what) {
      std::ostringstream o;
      o << "call " << n << " (" << c.form << " I=" << c.I << " T=" << c.T << "): " << what;
      return o.str();
    };
    if (c.form == "pieces") {
      fill((size_t)c.I * 512, (size_t)c.T * 512);
      continue;
    }
    if (c.form == "low") {
      fill(c.base, mlp_h_bytes(c.I, c.T));
      continue;
    }
    if (c.form == "plain") {
      fill(c.base + kMlpHOffset, mlp_h_bytes(c.I, c.T));
      continue;
    }
    uint64_t* ctl = &mem.at((c.base + kMlpCtlOffset) / 8);
    const int wgs = int(c.I / 16 + c.E / 16);
    clock += 500;  // 5 us at 100 MHz, less than any launch takes
    bool whole = ctl_is_signature(ctl[0]);
    for (int i = 0; i < kCtlMarks; ++i) whole = whole && ctl[ctl_mark(i)] == ctl_mark_value(ctl[0], i);
    if (!whole) {  // (one wave does it, the others wait for it)
      const uint64_t sig = ctl_signature(clock);
      for (int i = 1; i < kCtlWords; ++i) ctl[i] = ctl_initial(i, sig);
      ctl[0] = sig;
    }
    std::vector<int> looks(wgs), leaves(wgs);
    for (int w = 0; w < wgs; ++w) looks[w] = leaves[w] = w;
    std::shuffle(looks.begin(), looks.end(), rng);
    std::shuffle(leaves.begin(), leaves.end(), rng);
    std::vector<bool> looked(wgs);
    std::vector<uint64_t> epoch(wgs);
    size_t li = 0;
    for (int w : leaves) {  // a workgroup looks before it leaves; a random share of the others does so earlier
      while (!looked[w]) {
        const int v = (rng() & 1) ? w : looks[li++ % wgs];
        if (looked[v]) continue;
        epoch[v] = ctl_epoch(ctl[ctl_counter(ctl_group(v))]);
        looked[v] = true;
      }
      ctl[ctl_counter(ctl_group(w))] += ctl_arrival(w, wgs);
      if (w == 0)
        for (int g = wgs; g < kCtlGroups; ++g) ctl[ctl_counter(g)] += kCtlArrivalOfNone;
    }
    for (int w = 0; w < wgs; ++w)
      if (epoch[w] != epoch[0]) return fail("the workgroups of the launch read different epochs");
    std::ostringstream name;
    name << c.form << ":" << c.I << ":" << c.E << ":" << c.T << ":" << c.base;
    if (!seen.insert({name.str(), epoch[0]}).second) return fail("an earlier launch of the same call had this epoch");
    // what the launch writes
    if (c.form == "words") {
      fill(c.base + tagged_offset(c.I, c.T), (size_t)(c.T * c.I * 8));
    } else {
      fill(c.base + kMlpHOffset, (size_t)(c.T * c.I * 2));
      fill(c.base + mlp_slot_offset(c.I, c.T), (size_t)(c.I / 16 * 8));
    }
  }
  return "ok";
}

int main() {
  std::mt19937_64 rng(12345);
  std::string line;
  while (std::getline(std::cin, line)) {
    std::vector<Call> calls;
    std::istringstream in(line);
    std::string word;
    while (in >> word) {
      for (auto& ch : word)
        if (ch == ':') ch = ' ';
      std::istringstream f(word);
      Call c{};
      f >> c.form >> c.I >> c.E >> c.T >> c.base;
      calls.push_back(c);
    }
    std::cout << play(calls, rng) << "\n";
  }
}
