"""The work that users of this library have it do, as cases for timing it: single any-precision products from
one activation row up to the 16 that one call takes, work lists of a decoder layer, and the large-batch entry
points, over the shapes and bit-widths of the benchmark configurations (paper_2402_10517_amd/inputs.py) and
ragged ones.

Matrices are quantised with an 8-bit parent (n = 8), uniform indices, per-row ascending N(0, sigma) centroid tables
and N(0, 1) activations, all binary16 like the benchmark's; every case is drawn from its seed alone.
"""
import torch

from paper_2402_10517_amd import binding as B

N_BITS = 8
SIGMA = 0.02
BIT_WIDTHS = (3, 4, 5, 6, 7, 8)
# (M, K) = (output rows, columns) of the seven matrices of a 7B-shaped decoder layer: q, k, v, o, gate, up, down
DECODER_LAYER = ((4096, 4096),) * 4 + ((11008, 4096),) * 2 + ((4096, 11008),)
# the three distinct shapes of that layer; the benchmark's headline list is each of them at every bit-width
HEADLINE_SHAPES = ((4096, 4096), (11008, 4096), (4096, 11008))


def _case(kind, M, K, b, batch, name=None):
    c = {"kind": kind, "M": M, "K": K, "b": b, "batch": batch}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest configuration: one activation row, where latency and the launch are all there is.
        _case("gemv", 512, 512, 8, 1, "gemv_512x512_b8"),
        # One token through an attention projection of a 7B model: the most ordinary call.
        _case("gemv", 4096, 4096, 4, 1, "gemv_4096x4096_b4"),
        # One token through the gate or up projection of a 70B model: the largest single product.
        _case("gemv", 28672, 8192, 5, 1, "gemv_28672x8192_b5"),
        # Two queries at once through the down projection of a 13B model (rows with a ragged end).
        _case("gemv", 5120, 13824, 6, 2, "gemv_5120x13824_b6_batch2"),
        # Sizes that no tile divides: an odd number of rows, columns a multiple of 32 only, five queries.
        _case("gemv", 4099, 2208, 7, 5, "gemv_4099x2208_b7_batch5"),
        # Eight queries through the down projection of a 70B model at the lowest precision.
        _case("gemv", 8192, 28672, 3, 8, "gemv_8192x28672_b3_batch8"),
        # The largest batch of a single product call, through the gate projection of a 7B model.
        _case("gemv", 11008, 4096, 4, 16, "gemv_11008x4096_b4_batch16"),
        # The benchmark's headline: concurrent queries of all precisions, 18 independent products in one call.
        _case("headline", 0, 0, 0, 1, "list_headline_mixed"),
        # One decoder layer for four queries that run at 4 bits: seven products in one call.
        _case("layer", 0, 0, 4, 4, "list_decoder_layer_b4_batch4"),
        # A short prompt (64 tokens) through the gate projection of a 7B model at full precision.
        _case("gemm", 11008, 4096, 8, 64, "gemm_11008x4096_b8_batch64"),
        # A prompt of 512 tokens through an attention projection of a 70B model.
        _case("gemm", 8192, 8192, 3, 512, "gemm_8192x8192_b3_batch512"),
        # The large-batch call of programs that may not allocate, with a batch that no tile divides.
        _case("gemm_static", 4096, 4096, 5, 33, "gemm_static_4096x4096_b5_batch33"),
    ]


def _spread(rng, lo, hi):
    """A whole number in lo..hi, uniform in its logarithm."""
    return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "gemv", "gemv", "headline", "layer", "gemm", "gemm", "gemm_static"])
    b = rng.choice(BIT_WIDTHS)
    if kind == "headline":
        return _case(kind, 0, 0, 0, rng.choice([1, 1, 2]))
    if kind == "layer":
        return _case(kind, 0, 0, b, rng.randint(1, 8))
    if kind == "gemv":
        batch = rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 7, 8, rng.randint(9, 16)])
        most = 28672 * 8192 * 5 // b
    elif kind == "gemm":
        batch = _spread(rng, 17, 512)
        most = 8192 * 8192
    else:
        batch = _spread(rng, 17, 256)
        most = 4096 * 4096                       # what the library's static array holds
    step = rng.choice([32, 256])                 # any multiple of 32 columns, or whole tiles of them
    while True:
        M, K = _spread(rng, 512, 28672), _spread(rng, 512 // step, 28672 // step) * step
        if M * K <= most:
            return _case(kind, M, K, b, batch)


def _products(case):
    """(M, K, b) of every product of a pass."""
    if case["kind"] == "headline":
        return [(M, K, b) for M, K in HEADLINE_SHAPES for b in BIT_WIDTHS]
    if case["kind"] == "layer":
        return [(M, K, case["b"]) for M, K in DECODER_LAYER]
    return [(case["M"], case["K"], case["b"])]


def _draw_matrix(gen, M, K, bits):
    idx = torch.randint(0, 1 << N_BITS, (M, K), generator=gen, device="cuda", dtype=torch.uint8)
    luts = {b: (torch.randn((M, 1 << b), generator=gen, device="cuda") * SIGMA).half().sort(dim=1).values for b in bits}
    return idx, luts


def _inputs(case, seed):
    """The matrices [(idx, luts)] and the products [(matrix number, b, x)] of a pass, on the device."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    matrices, products = [], []
    numbers = {}
    for M, K, b in _products(case):
        shared = case["kind"] == "headline"      # one stored matrix serves every bit-width
        if shared and (M, K) in numbers:
            m = numbers[(M, K)]
        else:
            m = numbers[(M, K)] = len(matrices)
            matrices.append(_draw_matrix(gen, M, K, BIT_WIDTHS if shared else [b]))
        x = torch.randn((case["batch"], K), generator=gen, device="cuda").half()
        products.append((m, b, x))
    return matrices, products


def prepare(case, seed):
    matrices, products = _inputs(case, seed)
    packed = [B.ap_pack(idx.cpu().numpy(), {b: t.cpu().numpy() for b, t in luts.items()}) for idx, luts in matrices]
    state = {"kind": case["kind"], "batch": case["batch"], "packed": packed}
    if case["kind"] in ("headline", "layer"):
        state["items"] = [(packed[m], b, x, torch.empty((case["batch"], packed[m].M), dtype=torch.float16, device="cuda"))
                          for m, b, x in products]
    else:
        state["pm"], (_, state["b"], state["x"]) = packed[0], products[0]
        if case["kind"] == "gemm":               # the workspace that a program keeps from call to call
            state["work"] = torch.empty(case["M"] * case["K"] * 2, dtype=torch.uint8, device="cuda")
        if case["kind"] == "gemm_static":
            state["y"] = torch.empty((case["batch"], case["M"]), dtype=torch.float16, device="cuda")
    return state


def run(state):
    kind = state["kind"]
    if kind == "gemv":
        return B.ap_gemv(state["pm"], state["b"], state["x"])
    if kind == "gemm":
        return B.ap_gemm(state["pm"], state["b"], state["x"], work=state["work"])
    if kind == "gemm_static":
        x, y = state["x"], state["y"]
        status = B.lib.ap_gemm_static(state["pm"].handle, state["b"], x.data_ptr(), y.data_ptr(), x.shape[0],
                                      torch.cuda.current_stream().cuda_stream)
        if status != B.AP_OK:
            raise B.ApError(status, "ap_gemm_static")
        return y
    if state["batch"] == 1:
        return B.ap_gemv_list(state["items"])
    return B.ap_gemv_list_batch(state["items"], state["batch"])


def work(case):
    """Index bits, the centroid tables of the bit-widths used, activations and outputs, each once."""
    n = case["batch"]
    products = _products(case)
    nbytes = sum(M * (2 << b) + n * (K + M) * 2 for M, K, b in products)
    if case["kind"] == "headline":               # a matrix used at several bit-widths is read by each of them
        nbytes += sum(M * K * b // 8 for M, K, b in products)
    else:
        nbytes += sum(M * K * case["b"] // 8 for M, K, _ in products)
    return {"bytes": nbytes, "flops": sum(2 * M * K * n for M, K, _ in products)}


def tolerance(case):
    # Outputs are binary16 of sums held in binary32.  The library is 2.1e-4 from exact() on every case (the rounding
    # of the result), and two implementations differ by a binary16 step (up to 2^-10) where a sum falls on the
    # other side of a rounding boundary: four times each.
    return {"rel": 8e-4, "max": 4e-3}


def exact(case, seed):
    matrices, products = _inputs(case, seed)
    out = []
    for m, b, x in products:
        idx, luts = matrices[m]
        M, K = idx.shape
        x64, lut = x.double(), luts[b].double()
        y = torch.empty((x.shape[0], M), dtype=torch.float64, device="cuda")
        rows = max(1, (1 << 25) // K)
        for r in range(0, M, rows):
            w = lut[r:r + rows].gather(1, (idx[r:r + rows] >> (N_BITS - b)).long())
            y[:, r:r + rows] = x64 @ w.t()
        out.append(y)
    return out if case["kind"] in ("headline", "layer") else out[0]
