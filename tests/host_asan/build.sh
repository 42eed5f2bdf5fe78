#!/bin/bash
# Builds the C-ABI library with AddressSanitizer on its host code only (device
# code is compiled as in the product build) and the harnesses asan_driver and asan_graphs.
# Output: tests/host_asan/_build/asan_driver, asan_graphs. Run them with
#   ASAN_OPTIONS=detect_leaks=0:verify_asan_link_order=0 tests/host_asan/_build/asan_driver
set -e
HERE=$(cd "$(dirname "$0")" && pwd)
ROOT=$(cd "$HERE/../.." && pwd)
OUT=$HERE/_build
mkdir -p "$OUT"
HIPCC=${HIPCC:-/opt/rocm/bin/hipcc}
FLAGS="-O1 -g -fPIC -std=c++17 --offload-arch=gfx950 -Xclang -target-feature -Xclang -packed-fp32-ops -Xarch_host -fsanitize=address -Xarch_host -fno-omit-frame-pointer -I$ROOT/include -I$ROOT/paper_1009_3308_amd/csrc"
SRCS="host_numerics.cpp nse_api.cpp legendre_table.hip synthesis.hip ring_fft.hip analysis.hip contract_lp.hip pair_legendre.hip ndf_adaptive.hip diagnostics.hip"
pids=""
for f in $SRCS; do
  "$HIPCC" -x hip $FLAGS -c "$ROOT/paper_1009_3308_amd/csrc/$f" -o "$OUT/${f%.*}.o" &
  pids="$pids $!"
done
for p in $pids; do wait $p; done
OBJS=""
for f in $SRCS; do OBJS="$OBJS $OUT/${f%.*}.o"; done
for d in asan_driver asan_graphs; do
  "$HIPCC" -x hip $FLAGS -c "$HERE/$d.cpp" -o "$OUT/$d.o"
  "$HIPCC" --offload-arch=gfx950 -Xarch_host -fsanitize=address $OBJS "$OUT/$d.o" -o "$OUT/$d"
  echo "built $OUT/$d"
done
