// Which launches of the 14-state kernel take its form with two waves per SIMD (host code).
//
// The parts of a problem wait for each other, so a set of launches that run side by side has to
// find places for its gangs.  At three waves per SIMD a compute unit holds three 16-knot
// workgroups; a workgroup of the two-waves form takes half of the registers, and beside it there
// is room for one more of either form.  Gangs of that form therefore shrink what an XCD holds for
// every other launch on it: gangs of 16, 16, 32 and 32 parts on four streams fill the 96 places
// of an XCD exactly, but with the two short ones in the two-waves form each gang can hold all its
// places but some and wait for the rest until the limit (TIMEOUT).  Even a gang of two parts does
// that to some mix that fitted before.  A problem of one part waits for nobody and always leaves
// its place, so it takes nothing from any mix: only such launches have the form.
//
// Measured on MI355X, three waves per SIMD / two, us per iteration: one problem of 16 knots 1.02 /
// 0.79, 512 of them 1.24 / 1.03; what the line costs: one problem of 128 knots (8 parts) 1.77 /
// 1.67, 64 of them 1.95 / 1.86.
#pragma once
#include <stdint.h>

namespace mpc {

// `max_parts`: workgroups of the launch's largest problem; `tasks`: its workgroups; `places`:
// workgroups resident at two waves per SIMD where they run (one XCD or the device).
inline bool two_waves_form(int max_parts, int64_t tasks, int64_t places) {
  return max_parts == 1 && tasks <= places;
}

}  // namespace mpc
