#!/bin/bash
# Compile tests/host_mock/$1.cpp and link it with the objects that build.sh
# left in _build/mock/ (everything but the entry-point driver) into
# _build/mock/$1; further arguments go to the linker.  Run from the
# repository root, after build.sh:
#   bash tests/host_mock/link.sh shapes -Wl,--wrap=hipEventElapsedTime
set -e
ROOT=$(pwd)
OUT=$ROOT/_build/mock
NAME=$1
shift
SAN="-fsanitize=address,undefined -fno-omit-frame-pointer -fno-sanitize-recover=undefined"
/opt/rocm/llvm/bin/clang++ -O1 -g -std=c++17 $SAN -D__HIP_PLATFORM_AMD__ -I /opt/rocm/include -I $ROOT/include \
  $ROOT/tests/host_mock/$NAME.cpp $OUT/standardize.o $OUT/syrk.o $OUT/colsolve.o $OUT/kkt.o $OUT/polish.o \
  $OUT/output.o $OUT/warm.o $OUT/dense.o $OUT/api.o $OUT/penalty.o $OUT/mock_hip.o $OUT/fatbin_stubs.o \
  "$@" -lpthread -o $OUT/$NAME
echo "built $OUT/$NAME"
