"""The rules by which the library picks a kernel: host functions of libmbconv, called without a GPU."""
import ctypes as C

from paper_2110_10802_amd import binding as B

INT, BOOL, OUT = C.c_int, C.c_bool, C.POINTER(C.c_int)


def rule(symbol, restype, *argtypes):
    f = getattr(B.load(), symbol)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


def plan(symbol, *argtypes):
    """A rule that also says how many parts there are (its last argument): that number, or None."""
    f = rule(symbol, BOOL, *argtypes, OUT)

    def call(*args):
        n = C.c_int(0)
        return n.value if f(*args, C.byref(n)) else None
    return call


def wgrad_kernel(bf16, Ma, Mb, N, HW):
    """Which kernel computes the weight gradient of Ma x Mb channels over N planes of HW pixels."""
    if plan("_ZN3mbk13x3_wgrad_planEbiiiiPi", BOOL, INT, INT, INT, INT)(bf16, Ma, Mb, N, HW):
        return "x3"
    swap = C.c_bool(False)
    if plan("_ZN3mbk13wgrad_cl_planEiiiiPbPi", INT, INT, INT, INT, C.POINTER(C.c_bool))(Ma, Mb, N, HW, C.byref(swap)):
        return "lt"
    return "rd"


def block_wgrad_kernels(s):
    """Of a block's projection and expansion conv."""
    bf16 = s.dtype == "bf16"
    return (wgrad_kernel(bf16, s.Cout, s.Cexp, s.N, s.Ho * s.Wo), wgrad_kernel(bf16, s.Cexp, s.Cin, s.N, s.H * s.W))


def xs_chunks(s):
    """Chunks of the expansion conv's small-launch kernel, or None where another one runs."""
    return plan("_ZN3mbk12xs_conv_planEiiiiiiPi", *6 * [INT])(s.N, s.Cexp, s.Cin, s.H * s.W, 0, 1)


def se_bwd_tiled(N, channels, squeezed):
    """Whether the SE backward's two steps are those with a workgroup per sixteen channels."""
    return rule("_ZN3mbk12se_bwd_tiledEiii", BOOL, INT, INT, INT)(N, channels, squeezed)


def bw_form(N, M, K, HW, backward):
    """How the bf16 convolution with resident weights takes an expansion conv (or a projection conv's data gradient): steps of
    the contraction, chunks of 64 pixels to a wavefront and pixels in the last chunk; None where another kernel runs."""
    pro, epi = (2, 0) if backward else (0, 1)
    sets = plan("_ZN3mbk12bw_conv_planEiiiiiiPi", *6 * [INT])(N, M, K, HW, pro, epi)
    if sets is None or rule("_ZN3mbk14wave_conv_kindEiii", INT, INT, INT, INT)(M, K, HW) or \
            plan("_ZN3mbk12xk_conv_planEbiiiiiPi", BOOL, *5 * [INT])(True, N, M, K, HW, pro) is not None:
        return None
    chunks = -(-N * HW // 64)
    return -(-K // 32), -(-chunks // (4 * sets)), (N * HW - 1) % 64 + 1
