"""MI355X-native FLARE token mixer (encode-decode low-rank attention) behind a C ABI.

`synth` draws the seeded synthetic workloads; `binding` marshals arguments into
libflare.so (hand-written HIP kernels for gfx950) through _native.so; `autograd` makes the two calls
a differentiable step (a native autograd node).  Importing the package loads nothing
native; the first call into `binding` does, and raises if the library is missing.
"""
__all__ = ["synth", "binding", "autograd"]
