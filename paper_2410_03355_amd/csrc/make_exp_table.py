"""Writes exp_table.h, computed with 60 decimal digits:
2^(j/128), j = 0..127, as pairs (hi, lo) of doubles with hi the double nearest to the value and lo the double
nearest to the remainder, and 2^(j/256), j = 0..255, as pairs (hi, rest) of bit patterns with hi the double nearest to
the value, j 2^44 taken off its bits, and rest the double nearest to the remainder divided by hi.
Run from this directory: python make_exp_table.py > exp_table.h"""
import struct
from decimal import Decimal, getcontext

getcontext().prec = 60
N = 128
M = 256
LN2 = Decimal(2).ln()


def bits(x):
    return struct.unpack("<Q", struct.pack("<d", x))[0]


print("// 2^(j/128) for j = 0..127 as hi + lo, hi the nearest double and lo the nearest double to the")
print("// remainder, and 2^(j/256) for j = 0..255 as hi (1 + rest), hi the nearest double: bit patterns, j 2^44 taken off")
print("// those of hi (written by make_exp_table.py; the tables of the table-driven fp64 exponentials).")
print("#pragma once")
print("")
print("#include <stdint.h>")
print("")
print("namespace lantern {")
print("")
print("constexpr int EXP_TABLE_N = %d;" % N)
print("constexpr int EXP_FINE_N = %d;" % M)
print("#if defined(__HIPCC__)")
print("#define LANTERN_EXP_TABLE_QUAL __device__")
print("#else")
print("#define LANTERN_EXP_TABLE_QUAL")
print("#endif")
print("static const LANTERN_EXP_TABLE_QUAL double EXP_TABLE_HILO[2 * EXP_TABLE_N] = {")
for j in range(N):
    v = (LN2 * Decimal(j) / Decimal(N)).exp()
    hi = float(v)
    lo = float(v - Decimal(hi))
    print("    %s, %s," % (hi.hex(), lo.hex()))
print("};")
print("static const LANTERN_EXP_TABLE_QUAL uint64_t EXP_FINE[2 * EXP_FINE_N] = {")
for j in range(M):
    v = (LN2 * Decimal(j) / Decimal(M)).exp()
    hi = float(v)
    rest = float((v - Decimal(hi)) / Decimal(hi))
    print("    0x%016xull, 0x%016xull," % (bits(hi) - (j << 44), bits(rest)))
print("};")
print("")
print("}  // namespace lantern")
