#!/bin/bash
# Builds libmoe_mi355x.so for gfx950, which needs ROCm alone, and then the Python layer's marshalling, which needs the headers of the
# Python ($PYTHON, default python3) and the torch that will load it and names them; without them it is left out, and binding.py does
# without.  (Run from anywhere; output lands next to the package.)
# -Wno-inline-asm: the LDS-DMA loads name M0 in their clobber list on purpose (they set it).
set -e
cd "$(dirname "$0")"
hipcc --offload-arch=gfx950 -O3 -std=c++17 -fPIC -shared \
  -Xclang -target-feature -Xclang -packed-fp32-ops -Wno-inline-asm "$@" \
  api.hip route.hip plan.hip rowmove.hip expert_f32.hip expert_bf16.hip expert_small.hip router.hip router_dx.hip router_dw.hip probes.hip alloc.hip -o ../libmoe_mi355x.so

if ! torch_flags=$("${PYTHON:-python3}" - <<'P'
import sys, sysconfig, torch
from torch.utils import cpp_extension as ext
lib = ext.library_paths()
print(*("-isystem " + p for p in ext.include_paths("cuda") + [sysconfig.get_paths()["include"]]), *("-L" + p for p in lib),
      *("-Wl,-rpath," + p for p in lib), f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
      f"-o ../_marshal.{sys.implementation.cache_tag}.torch-{torch.__version__}.so")
P
) || ! g++ -O2 -std=c++17 -fPIC -shared -D__HIP_PLATFORM_AMD__=1 -DUSE_ROCM=1 marshal.cpp -ltorch_python -ltorch_cpu -lc10 -lc10_hip $torch_flags
then echo "the native marshalling was not built: the Python layer will check its arguments itself" >&2
fi
