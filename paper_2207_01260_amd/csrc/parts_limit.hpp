// When a block on three bf16 parts (mbrow3_kernel.hpp) has to run on the fp32 instruction, from the largest magnitudes of its weights.
//
// A number below 2^-110 loses at most 2^-134 as three parts (half of bf16's last bit).  A final sum that is below 2^-50 and not zero is
// made again, so what was lost must be below half the last place of 2^-50, 2^-75, by the time it gets there.  With n1 terms of the
// expansion, n2 of the projection, Mx, Me, Md, Mp the largest input and weights, D the largest depthwise result:
//   an input's loss      n1 Me 9 Md n2 Mp 2^-134  <  2^-75      an expansion weight's    n1 Mx 9 Md n2 Mp 2^-134  <  2^-75
//   a depthwise result's              n2 Mp 2^-134  <  2^-75      a projection weight's                n2 D 2^-134  <  2^-75
// Those on the left depend on weights only.  Those on the right matter where there is a weight that small, which trained networks have
// (filters that died): Mx, or D, is then limited, and weights of ordinary size leave both limits far above ordinary activations.
// Infinities and NaN among the weights fail every comparison.  2^60: with inputs and expansion weights below it no product overflows.
#pragma once
#include <stdint.h>
#include <string.h>
#include "cprune.h"
#include "split_index.hpp"

namespace cprune {

// p: n1 = p.terms, n2 = p.cpe and the activations; me ... mp, be, bd: largest magnitudes; small_e, small_p: there is a weight that is not
// zero and below 2^-110
template <typename P>
CPRUNE_HD uint32_t parts_limit(const P& p, float me, float md, float mp, float be, float bd, bool small_e, bool small_p) {
  const double room = 0x1p58, n1 = p.terms, n2 = p.cpe;      // a bit less than the 2^59 above
  double limit;
  if (p.we) {
    const double gain = n2 * mp * 9.0 * md;                  // of an expanded number, in a final sum
    limit = 0x1p60;
    if (!(me < 0x1p60f) || !(n1 * me * gain <= room) || !(n2 * mp <= room)) return 0;
    auto at_most = [&](double v) { if (!(limit <= v)) limit = v; };
    if (small_e && gain > 0.0) at_most(room / (n1 * gain));
    if (small_p && p.act_d != CPRUNE_ACT_RELU6) {
      if (p.act_e == CPRUNE_ACT_RELU6) {
        if (!(n2 * (54.0 * md + bd) <= room)) return 0;
      } else if (md > 0.0f && me > 0.0f) {
        at_most(((room / n2 - bd) / (9.0 * md) - be) / (n1 * me));
      }
    }
    if (!(limit > 0.0)) return 0;
  } else {
    // (fewer than 16 terms, and every weight too large: always)
    if (p.ce < 16 || !(n2 * mp <= room)) return 0;
    if (!small_p || p.act_d == CPRUNE_ACT_RELU6) return 0xffffffffu;
    limit = room / n2;
  }
  const float f = (float)limit;
  uint32_t bits;
  memcpy(&bits, &f, 4);
  return p.we ? bits >> 16 : bits;
}

}  // namespace cprune
