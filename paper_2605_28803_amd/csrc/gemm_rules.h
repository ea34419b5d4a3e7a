// Index arithmetic of the products that has to hold for every size, in plain
// C++ (no HIP), so that it can be checked on the host.
#pragma once

namespace oq {

// The few-row product walks K in units of 128 codes (64 packed bytes of a row;
// 128 bytes of 8-bit codes), nu = K / 128 of them.  Wave `wave` of `waves`
// takes units [small_begin(wave), small_begin(wave + 1)).
constexpr int small_begin(int nu, int wave, int waves) { return (nu * wave) / waves; }

// The unit that is loaded where unit u of a wave that ends at uend is asked
// for: loads are unconditional, and one past the end reads unit uend - 1 or 0
// again.
constexpr int small_unit(int u, int uend) { return u < uend ? u : uend > 0 ? uend - 1 : 0; }

// Byte within a unit that a quarter wave reads 16 bytes at (8-bit codes: twice
// that, 32 bytes).  At K = 64 there is no whole unit: rows hold half of one,
// and every quarter stays in that half (nothing loaded there is used).
constexpr int small_piece(int nu, int quarter) { return 16 * (nu > 0 ? quarter : quarter & 1); }

}  // namespace oq
