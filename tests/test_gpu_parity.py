"""GPU parity: the HIP path through the C ABI against the CPU oracle.

Integer outputs (active set, |S|, remapped labels) must match bit for bit;
floating point within the stated bar and the derived bounds of _gpu_util.
Sizes span several tiles of every kernel and leave ragged tails in the batch
and in |S|.
"""

import numpy as np
import pytest
import torch

import workloads
from oracle import pfc_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2010_05222_amd import pfc  # noqa: F401  (fails loudly if libpfc.so is missing)
    return torch.device("cuda:0")


def _shard(B, d, C, r, dtype, margin, m, class_offset=0, dev="cuda:0", tau=None):
    from paper_2010_05222_amd.head import PfcShard
    return PfcShard(B, d, C, r, dtype=dtype, class_offset=class_offset, s=64.0, m=m,
                    margin=margin, lr=0.1, mu=0.9, device=dev, tau=tau)


def _case(dev, B, d, C, r, dtype, margin, m, seed, class_offset=0, label_span=None,
          random_m=True, master=False, labels=None, tau=None, conflicts=0, abs_scaled=False,
          degenerate=False):
    from _gpu_util import make_problem, run_and_compare
    print(f"\ncase B={B} d={d} C={C} r={r} dtype={dtype} margin={margin} seed={seed} "
          f"offset={class_offset} master={master} tau={tau}", flush=True)
    Xd, Wd, Md, Pd, Ld = make_problem(B, d, C, dtype, seed, class_offset, label_span, random_m,
                                      master, labels, dev, conflicts)
    shard = _shard(B, d, C, r, dtype, margin, m, class_offset, dev, tau)
    out = run_and_compare(shard, Xd, Wd, Md, Pd, Ld, seed, margin, abs_scaled=abs_scaled,
                          degenerate=degenerate)
    print(out, flush=True)
    return out


def test_tiny_workload_fp32(dev):
    """The parity-scale workload (B=64, d=128, C=10,000, r=0.1, fp32, CosFace)."""
    cfg = workloads.config("tiny")
    from _gpu_util import run_and_compare
    X, labels = workloads.make_batch(cfg, 0)
    W = workloads.make_weights_host(cfg)
    Xd = torch.from_numpy(X).to(dev)
    Wd = torch.from_numpy(W).to(dev)
    Ld = torch.from_numpy(labels).to(dev)
    for random_m in (False, True):
        Md = torch.from_numpy(workloads.make_momentum_host(cfg, random=random_m)).to(dev)
        shard = _shard(cfg["B"], cfg["d"], cfg["C"], cfg["r"], "f32", cfg["margin"], cfg["m"],
                       dev=dev)
        out = run_and_compare(shard, Xd, Wd.clone(), Md, None, Ld, 0, cfg["margin"])
        assert out["K"] == 1000
        print(out, flush=True)


@pytest.mark.parametrize("margin,m", [("cosface", 0.4), ("arcface", 0.5)])
def test_bf16_ragged(dev, margin, m):
    # B not a multiple of any tile; |S| = 300 not a multiple of 32/64/128.
    _case(dev, 100, 128, 3000, 0.1, "bf16", margin, m, seed=1)


def test_bf16_master(dev):
    _case(dev, 96, 256, 4000, 0.2, "bf16", "arcface", 0.5, seed=2, master=True)


def test_f16_ragged(dev):
    _case(dev, 70, 256, 5000, 0.2, "f16", "arcface", 0.5, seed=3)


def test_bf16_d512_several_tiles(dev):
    _case(dev, 300, 512, 20000, 0.1, "bf16", "cosface", 0.4, seed=4, random_m=False)


def test_f16_d512_zero_momentum(dev):
    _case(dev, 260, 512, 12000, 0.1, "f16", "arcface", 0.5, seed=5, random_m=False)


def test_f16_d512_master(dev):
    # fp16 weights with an fp32 master at d = 512; |S| = 910, B ragged.
    _case(dev, 190, 512, 9100, 0.1, "f16", "cosface", 0.4, seed=18, master=True)


def test_f16_d128(dev):
    _case(dev, 150, 128, 4100, 0.1, "f16", "cosface", 0.4, seed=19)


@pytest.mark.parametrize("d", [8, 1000, 1024])
def test_f32_feature_widths(dev, d):
    # The fp32 path takes any d that is a multiple of 8 up to 1024: the
    # smallest, one that is not a multiple of 32 or 64, and the largest.
    # At d = 8 the class rows (std 0.01) have norm ~0.028, so 1/||w|| ~ 35
    # and the class gradients reach ~72, where one fp32 ulp is 7.6e-6: the
    # max-abs bar is applied relative to max |ref| there (as for B = 1);
    # the row-relative bound is unchanged.
    _case(dev, 40, d, 1500, 0.2, "f32", "arcface", 0.5, seed=27, abs_scaled=(d == 8))


@pytest.mark.parametrize("B,d,C,r,master,tau", [
    (1, 8, 40, 0.5, False, None),          # one row, one 64-column block, a partial class tile
    (16, 64, 330, 0.1, True, None),        # a full 16-row wave; |S| = 33
    (65, 520, 640, 0.1, False, 0.4),       # one row past a 64-row tile; nine column blocks
    (33, 1016, 650, 0.1, True, None),      # 32 + 1 rows of dX; sixteen column blocks, |S| = 65
    (600, 200, 8200, 0.5, False, 0.4),     # enough tiles for the 64-class forward
])
def test_f32_tile_edges(dev, B, d, C, r, master, tau):
    # The max-abs bar relative to max |ref|: the gradient scale s/B is 64 / B.
    _case(dev, B, d, C, r, "f32", "arcface", 0.5, seed=61, master=master, tau=tau, conflicts=2,
          abs_scaled=True)


def test_f32_rows_need_no_16_byte_alignment(dev):
    """fp32 tensors that start 4 bytes past a 16-byte boundary give the aligned
    ones' results bit for bit."""
    from _gpu_util import make_problem
    outs = []
    for off in (0, 1):
        parts = make_problem(40, 136, 900, "f32", 62, master=True, device=dev)
        Xd, Wd, Md, Pd = (torch.empty(t.numel() + 4, device=dev)[off:off + t.numel()]
                          .view_as(t).copy_(t) for t in parts[:4])
        assert Xd.data_ptr() % 16 == 4 * off
        shard = _shard(40, 136, 900, 0.2, "f32", "arcface", 0.5, dev=dev)
        shard.dX = torch.empty(40 * 136 + 4, device=dev)[off:off + 40 * 136].view(40, 136)
        shard.step(Xd, parts[4], Wd, Md, 62, Pd)
        torch.cuda.synchronize()
        outs.append((shard.loss, shard.row_lse, shard.dX, Xd, Wd, Md, Pd))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,d,K,dtype", [
    (70, 128, 1500, "f16"), (70, 256, 1500, "bf16"), (70, 512, 1500, "bf16"),   # 64-row tiles, if aligned
    (513, 256, 8192, "bf16"),                                                   # 256-row tiles
])
def test_16_bit_batch_needs_no_16_byte_alignment(dev, B, d, K, dtype):
    """Embeddings that start 2 or 8 bytes past a 16-byte boundary give the
    aligned ones' results bit for bit."""
    from _gpu_util import make_problem
    Xd, Wd, Md, _, Ld = make_problem(B, d, K, dtype, 72, device=dev)
    outs = []
    for off in (0, 1, 4):
        print(f"\nbatch alignment: B={B} d={d} K={K} {dtype} offset {off}", flush=True)
        X = torch.empty(Xd.numel() + 8, dtype=Xd.dtype, device=dev)[off:off + Xd.numel()]
        X = X.view_as(Xd).copy_(Xd)
        assert X.data_ptr() % 16 == 2 * off
        W, M = Wd.clone(), Md.clone()
        shard = _shard(B, d, K, 1.0, dtype, "arcface", 0.5, dev=dev)
        shard.step(X, Ld, W, M, 72)
        torch.cuda.synchronize()
        outs.append((shard.loss, shard.row_lse, shard.dX, W, M))
    for out in outs[1:]:
        for x, y in zip(out, outs[0]):
            assert torch.equal(x, y)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_single_class_shard(dev, dtype):
    # The smallest shard: one class, taken at r = 1.  Rows labelled with it
    # have a one-term softmax (probability 1, loss 0, no gradient); the
    # others are unowned and their only logit gets the full gradient, so the
    # class gradient reaches ~30.  References that are exactly zero and that
    # magnitude take the degenerate-case and scaled bars.
    labels = np.array([0, 3, 0, 9, 0, 0, 5, 0, 2, 0, 0, 4])
    out = _case(dev, 12, 128, 1, 1.0, dtype, "arcface", 0.5, seed=28, labels=labels,
                abs_scaled=True, degenerate=True)
    assert out["K"] == 1


def test_positives_exceed_budget(dev):
    out = _case(dev, 512, 128, 1000, 0.05, "bf16", "cosface", 0.4, seed=6)
    assert out["K"] == out["n_pos"] > 50


def test_r1_full_softmax(dev):
    out = _case(dev, 64, 128, 2000, 1.0, "bf16", "arcface", 0.5, seed=7)
    assert out["K"] == 2000


def test_unowned_labels_and_offset(dev):
    # Shard [1000, 3000) of a larger head; a third of the labels fall outside it.
    _case(dev, 128, 128, 2000, 0.1, "bf16", "arcface", 0.5, seed=8, class_offset=1000,
          label_span=(0, 4000))


def test_no_owned_labels(dev):
    _case(dev, 32, 128, 2000, 0.1, "bf16", "cosface", 0.4, seed=9, class_offset=5000,
          label_span=(0, 4000))


def test_duplicated_positives(dev):
    rng = np.random.default_rng(10)
    labels = rng.choice(np.array([3, 17, 17, 17, 250, 999]), size=200)
    _case(dev, 200, 128, 1000, 0.1, "bf16", "cosface", 0.4, seed=10, labels=labels)


def test_single_row_and_tiny_shard(dev):
    # B = 1 makes the gradient scale s/B = 64, so |g| reaches ~100 here, two
    # orders of magnitude above any workload's.  The bf16 coefficients carry
    # ~2^-9 relative error, so the max-abs bar is applied relative to the
    # reference magnitude (max(1, max |ref|) times the stated bar) in this
    # case only; the row-relative bound is unchanged.
    _case(dev, 1, 128, 7, 0.5, "bf16", "arcface", 0.5, seed=11, abs_scaled=True)


def test_repeat_is_deterministic(dev):
    """Same inputs twice: bit-identical outputs (no floating-point atomics)."""
    from _gpu_util import make_problem
    outs = []
    for _ in range(2):
        Xd, Wd, Md, Pd, Ld = make_problem(200, 256, 6000, "bf16", 12, device=dev)
        shard = _shard(200, 256, 6000, 0.1, "bf16", "arcface", 0.5, dev=dev)
        shard.step(Xd, Ld, Wd, Md, 12)
        torch.cuda.synchronize()
        outs.append((shard.loss.clone(), shard.dX.clone(), Wd.clone(), Md.clone()))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("name", ["one_shard", "zipf", "massive"])
def test_sampler_full_size(dev, name):
    """Bit-exact active set and remap at the workloads' full shard sizes."""
    cfg = workloads.config(name)
    _, labels = workloads.make_batch(cfg, 0)
    print(f"\nsampler {name}: B={cfg['B']} C={cfg['C']} r={cfg['r']}", flush=True)
    shard = _shard(cfg["B"], cfg["d"], cfg["C"], cfg["r"], cfg["dtype"], cfg["margin"], cfg["m"],
                   dev=dev)
    Ld = torch.from_numpy(labels).to(dev)
    shard.sample(Ld, 0)
    torch.cuda.synchronize()
    active_ref, mapped_ref, info = O.sample_active(labels, cfg["C"], cfg["a"], cfg["r"], 0)
    K = int(shard.n_active.item())
    assert K == len(active_ref) == max(O.budget(cfg["r"], cfg["C"]), info["n_pos"])
    assert np.array_equal(shard.active[:K].cpu().numpy(), active_ref)
    assert np.array_equal(shard.labels_mapped.cpu().numpy(), mapped_ref)


# Shards that do not start on a Philox block (class_offset not a multiple of
# four), ragged last groups, every selection mode (keys; all classes at r = 1;
# positives only when they exceed the budget), duplicated and unowned labels.
@pytest.mark.parametrize("B,C,a,r,seed", [
    (64, 9001, 3, 0.1, 21),
    (300, 70001, 1000001, 0.05, 22),
    (8, 17, 2, 0.5, 23),
    (256, 5000, 6, 0.01, 24),       # |P| > budget: positives only
    (40, 2003, 5, 1.0, 25),         # every class
    (1000, 12289, 4097, 0.3, 26),   # most labels in one 4,096-class group
    (64, 9001, 2**40 + 3, 0.1, 29), # global ids above 2^32: the counter's high word
])
def test_sampler_offsets_and_modes(dev, B, C, a, r, seed):
    rng = np.random.default_rng(seed)
    labels = rng.integers(max(a - 50, 0), a + C + 50, size=B)  # some outside the shard
    if C > 8192:
        labels[: B // 2] = rng.integers(a + 4096, a + 8192, size=B // 2)
    labels[::7] = labels[0]                                    # duplicates
    print(f"\nsampler B={B} C={C} a={a} r={r} seed={seed}", flush=True)
    shard = _shard(B, 128, C, r, "bf16", "arcface", 0.5, class_offset=a, dev=dev)
    shard.sample(torch.from_numpy(labels.astype(np.int64)).to(dev), seed)
    torch.cuda.synchronize()
    active_ref, mapped_ref, info = O.sample_active(labels, C, a, r, seed)
    K = int(shard.n_active.item())
    assert K == len(active_ref) == max(O.budget(r, C), info["n_pos"])
    assert np.array_equal(shard.active[:K].cpu().numpy(), active_ref)
    assert np.array_equal(shard.labels_mapped.cpu().numpy(), mapped_ref)


def _sampler_case(dev, labels, C, a, r, seed):
    print(f"\nsampler B={len(labels)} C={C} a={a} r={r} seed={seed}", flush=True)
    shard = _shard(len(labels), 128, C, r, "bf16", "arcface", 0.5, class_offset=a, dev=dev)
    shard.sample(torch.from_numpy(labels.astype(np.int64)).to(dev), seed)
    torch.cuda.synchronize()
    active_ref, mapped_ref, info = O.sample_active(labels, C, a, r, seed)
    K = int(shard.n_active.item())
    assert K == len(active_ref) == max(O.budget(r, C), info["n_pos"])
    assert np.array_equal(shard.active[:K].cpu().numpy(), active_ref)
    assert np.array_equal(shard.labels_mapped.cpu().numpy(), mapped_ref)
    return info


@pytest.mark.parametrize("C,a,r", [
    (4096, 0, 0.5), (4097, 1, 0.5),                  # one group, one class past it
    (1 << 20, 0, 0.1), ((1 << 20) + 1, 3, 0.1),      # one group per workgroup, two
    (1 << 21, 0, 0.01), ((1 << 21) + 1, 2, 0.01),    # threshold found per workgroup, once
    (3000, 0, 2999 / 3000),                          # all but one
])
@pytest.mark.parametrize("B", [1, 8192])
def test_sampler_group_edges(dev, B, C, a, r):
    rng = np.random.default_rng(63)
    labels = rng.integers(a, a + C, size=B)
    labels[1::3] = np.iinfo(np.int64).min + 1   # no class of any shard
    _sampler_case(dev, labels, C, a, r, 64)


@pytest.mark.parametrize("B,C,a,r", [
    (128, 3000001, 1, 0.1),           # above 512 groups, candidates held in LDS
    (8192, 8000001, 2, 0.5),          # 22,300 candidates: held
    (64, 8192 * 4096, 0, 0.001),      # the most groups whose candidates are held
    (64, 8192 * 4096 + 1, 3, 0.001),
])
def test_sampler_above_512_groups(dev, B, C, a, r):
    labels = np.random.default_rng(70).integers(a - 1, a + C + 1, size=B)
    _sampler_case(dev, labels, C, a, r, 71)


@pytest.mark.parametrize("C,b,seed", [
    (1000, 1, 4572), (9001, 1, 60), (1100003, 1, 2488), (2200003, 1, 4342),
    (100, 99, 10856), (2200003, 2200002, 413),
])
def test_sampler_threshold_outside_window(dev, C, b, seed):
    """Seeds whose threshold lies outside the window in which the sampler
    expects it (five standard deviations and four classes around the budget):
    it is then found over all keys."""
    from oracle import philox
    labels = np.array([C + 5])                       # unowned: b negatives
    slack = 5.0 * np.sqrt(b * (1 - b / C)) + 4.0
    key = np.partition(philox.class_keys(seed, np.arange(C)), b - 1)[b - 1]
    at = float(key) / 2.0 ** 64 * C
    assert at < b - 1 - slack or at > b + slack
    _sampler_case(dev, labels, C, 0, b / C, seed)


@pytest.mark.parametrize("B,C,b,seed", [
    (5000, 13001, 13000, 1), (4000, 16385, 16384, 1), (2000, 61282, 61281, 2),
    (8192, 2200003, 2200002, 0),
])
def test_sampler_threshold_in_the_last_bin(dev, B, C, b, seed):
    """A budget that leaves one class out of a shard with many positives: the
    window of candidates ends with the last key, and the threshold lies in a
    bin of it that would end past 2^64."""
    from oracle import philox
    labels = np.random.default_rng(seed).integers(0, C + C // 4, size=B)
    slack = 5.0 * np.sqrt(b * (1 - b / C)) + 4.0
    lo = int(max(0.0, (b - min(B, C) - slack) / C * 2.0 ** 32)) << 32
    shift = (2 ** 64 - 1 - lo).bit_length() - 11
    keys = philox.class_keys(seed, np.arange(C))
    keep = keys >= np.uint64(lo)
    keep[labels[labels < C]] = False
    threshold = int(np.sort(keys[keep])[b - C - 1])
    assert lo + ((((threshold - lo) >> shift) + 1) << shift) > 2 ** 64
    _sampler_case(dev, labels, C, 0, b / C, seed)


def _candidates(labels, C, a, r, seed):
    """Non-positive keys inside the sampler's window (five standard deviations
    and four classes around where the threshold can lie), and its groups of
    4,096 classes."""
    from oracle import philox
    b = O.budget(r, C)
    slack = 5.0 * np.sqrt(b * (1 - b / C)) + 4.0
    lo = max(0.0, (b - min(len(labels), C) - slack) / C * 2.0 ** 32)
    hi = min(2.0 ** 32 - 1, np.ceil((b + slack) / C * 2.0 ** 32))
    top = philox.class_keys(seed, np.arange(a, a + C)) >> np.uint64(32)
    inside = (top >= np.uint64(int(lo))) & (top <= np.uint64(int(hi)))
    own = labels[(labels >= a) & (labels < a + C)] - a
    inside[own] = False
    return int(np.count_nonzero(inside)), -(-C // 4096)


@pytest.mark.parametrize("B,C,r,most,groups", [
    (8192, 1_000_000, 0.5, 8192, (5, 512)),           # each writing workgroup's list
    (8192, 20_000_000, 0.5, 28672, (513, 8192)),      # the resolving workgroup's
])
def test_sampler_candidates_beyond_lds(dev, B, C, r, most, groups):
    """More candidates than the kernel that finds the threshold holds in LDS: it
    reads them from memory for each pass."""
    labels = np.random.default_rng(31).integers(0, C, size=B)
    n, n_groups = _candidates(labels, C, 0, r, 31)
    assert n > most and groups[0] <= n_groups <= groups[1], (n, n_groups)
    _sampler_case(dev, labels, C, 0, r, 31)


def test_sampler_20m_classes(dev):
    labels = np.random.default_rng(31).integers(0, 20_000_000, size=1024)
    _sampler_case(dev, labels, 20_000_000, 0, 0.01, 31)


def test_many_rows_per_class(dev):
    # Every row is labelled with one of three classes of the same 128-class
    # tile: each quarter of the batch holds more target rows of that tile than
    # the class-gradient kernel lists, so it scans the labels instead.
    rng = np.random.default_rng(13)
    labels = rng.choice(np.array([5, 6, 100]), size=2400)
    _case(dev, 2400, 128, 3000, 0.1, "bf16", "arcface", 0.5, seed=13, labels=labels)


@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (256, "f16"), (512, "bf16")])
@pytest.mark.parametrize("B,C,r", [
    (5, 90, 0.4),        # two 32-class chunks: two splits, one run of them
    (385, 6000, 0.3),    # four row blocks of 128, one of a single row; 57 chunks
    (129, 40000, 0.5),   # more chunks than splits
])
def test_feature_gradient_splits(dev, B, C, r, d, dtype):
    # Splits of the class range and the runs that sum them.  The max-abs bar
    # relative to max |ref|: the gradient scale is 64 / B.  At d = 128 logits
    # spread by 64 / sqrt(128) = 5.7, and of 20,000 classes a few have all 129
    # softmax numerators below 2^-14 of their group's maximum, where the fp16
    # store's steps of 2^-24 are no longer 2^-11 of them (a class gradient row
    # off by 4 %): 3,600 classes there.
    if d == 128 and C == 40000:
        C, r = 12000, 0.3
    _case(dev, B, d, C, r, dtype, "arcface", 0.5, seed=65, random_m=False, abs_scaled=True)


@pytest.mark.parametrize("d,dtype,master", [(128, "bf16", True), (256, "f16", False),
                                            (512, "bf16", True), (512, "f16", False)])
def test_class_tiles_agree(dev, d, dtype, master):
    """The class-gradient tiles of 128, 64 and 32 classes give a class the same
    momentum row bit for bit.  A shard of more than a round of 128-class tiles, against
    shards of some of its classes (whole 128-class groups), whose tiles are
    others, given its row log-sum-exp."""
    from _gpu_util import make_problem
    # One row tile of 64 (so that every shard's forward is the narrow one).
    B, n_cu = 60, torch.cuda.get_device_properties(dev).multi_processor_count
    C = 128 * n_cu + 66 * 128 + 33
    Xd, Wd, Md, Pd, Ld = make_problem(B, d, C, dtype, 66, master=master, device=dev)
    Ld[3:9] = Ld[2]                             # rows of one class

    def run(lo, hi, lse):
        print(f"\nclass tiles: d={d} {dtype} classes [{lo}, {hi})", flush=True)
        W, M = Wd[lo:hi].clone(), Md[lo:hi].clone()
        P = Pd[lo:hi].clone() if master else None
        shard = _shard(B, d, hi - lo, 1.0, dtype, "arcface", 0.5, class_offset=lo, dev=dev)
        shard.sample(Ld, 0)
        shard.forward(Xd, W)
        shard.backward(Xd, W, M, P, row_lse=shard.row_lse if lse is None else lse)
        torch.cuda.synchronize()
        return shard.row_lse.clone(), W, M, P

    lse, W, M, P = run(0, C, None)
    full = 128 * n_cu
    for lo, hi in [(0, 128), (full - 128, C), (0, 128 * (n_cu // 4)), (256, 256 + 128 * 129),
                   (full, C), (0, 128 * (n_cu // 2)), (0, full), (128, full + 256)]:
        _, w, m, p = run(lo, hi, lse)
        assert torch.equal(m, M[lo:hi])
        assert p is None or torch.equal(p, P[lo:hi])
        # The same fp32 step, rounded to the storage type once, or (where the
        # compiler fuses the step's last operation with the conversion to fp16)
        # without the fp32 rounding before: at most one unit in the last place.
        ulp = 2.0 ** -10 if dtype == "f16" else 0.0
        assert torch.all((w.float() - W[lo:hi].float()).abs() <= ulp * W[lo:hi].float().abs())


@pytest.mark.parametrize("B,d,K,dtype,tau", [
    (512, 256, 8192, "f16", 0.4),     # 512 narrow forward tiles (64 rows), the most they are used for
    (513, 256, 8192, "f16", 0.4),     # one row tile more: the 256-row kernel
    (64, 512, 65409, "bf16", None),   # 512 class tiles, one class in the last: narrow
    (65, 512, 32769, "bf16", 0.4),    # 257 class tiles of two row tiles each: the 256-row kernel
])
def test_forward_tile_widths(dev, B, d, K, dtype, tau):
    """Both forward kernels around the line between them: ragged tiles, the
    PFC* filter, rows whose label is outside the shard."""
    _case(dev, B, d, K, 1.0, dtype, "arcface", 0.5, seed=67, class_offset=100,
          label_span=(0, K + 200), tau=tau, conflicts=4, random_m=False)


@pytest.mark.parametrize("dtype,d,tau", [("bf16", 512, None), ("f16", 128, 0.4), ("f32", 200, None),
                                         ("f32", 512, 0.4)])
def test_forward_tiles_agree(dev, dtype, d, tau):
    """A row's log-sum-exp does not depend on the tiles that its batch takes:
    64 rows of a batch of 600 (the 256-row forward kernel; in fp32 the 64-class
    tiles), alone (the narrow kernel; 32-class tiles), give the same bits."""
    from _gpu_util import make_problem
    B, C, lo = 600, 8000, 128
    Xd, Wd, _, _, Ld = make_problem(B, d, C, dtype, 68, label_span=(0, C + 900), device=dev,
                                    conflicts=4)
    out = []
    for rows in (slice(0, B), slice(lo, lo + 64)):
        X, L = Xd[rows].contiguous(), Ld[rows].contiguous()
        shard = _shard(len(X), d, C, 1.0, dtype, "arcface", 0.5, dev=dev, tau=tau)
        shard.sample(L, 0)
        shard.forward(X, Wd)
        out.append(shard.row_lse)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out[0]).all())
    assert torch.equal(out[0][lo:lo + 64], out[1])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_row_merges_agree(dev, dtype):
    """A row's log-sum-exp does not depend on the form of the row merge that its
    batch takes: 4,096 rows at once (one wave per row), and by 1,024, 256 and
    128 of them (four waves per row), give the same bits.  Scale 1, so that all
    of a row's 430 tiles count in its sum."""
    from _gpu_util import make_problem
    B, d, C = 4096, 128, 55000
    Xd, Wd, _, _, Ld = make_problem(B, d, C, dtype, 73, device=dev)
    out = []
    for rows in (4096, 1024, 256, 128):
        print(f"\nrow merges: {dtype} batches of {rows}", flush=True)
        shard = _shard(rows, d, C, 1.0, dtype, "arcface", 0.5, dev=dev)
        shard.s = 1.0
        lse = []
        for k in range(0, B, rows):
            shard.sample(Ld[k:k + rows].contiguous(), 0)
            shard.forward(Xd[k:k + rows].contiguous(), Wd)
            lse.append(shard.row_lse.clone())
        out.append(torch.cat(lse))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out[0]).all())
    for lse in out[1:]:
        assert torch.equal(out[0], lse), int((out[0] != lse).sum())


@pytest.mark.parametrize("dtype,d,tau", [("bf16", 512, None), ("f16", 128, 0.4), ("bf16", 256, 0.4)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_centre_reaches_every_row(dev, dtype, d, tau, bad):
    """A class centre with a NaN or an infinity has a NaN cosine to every row,
    so each row's log-sum-exp and the loss are NaN, in both forward kernels and
    also in the rows that are labelled with the class."""
    from _gpu_util import make_problem
    B, C, c = 600, 8000, 4321
    Xd, Wd, _, _, Ld = make_problem(B, d, C, dtype, 69, device=dev)
    Ld[130:190:7] = c
    Wd[c, 3] = bad
    for rows in (slice(0, B), slice(128, 192)):       # 256-row tiles; 64-row tiles
        X, L = Xd[rows].contiguous(), Ld[rows].contiguous()
        print(f"\nnon-finite centre: {dtype} d={d} tau={tau} {bad} rows {rows}", flush=True)
        shard = _shard(len(X), d, C, 1.0, dtype, "arcface", 0.5, dev=dev, tau=tau)
        shard.sample(L, 0)
        shard.forward(X, Wd)
        torch.cuda.synchronize()
        assert bool(torch.isnan(shard.row_lse).all())
        assert bool(torch.isnan(shard.loss).all())


# PFC* conflict filter (Sec. 3.3.4, Eq. noise_filtering): some rows sit near
# the centre of another row's class, so their cosine to that (active)
# negative is ~0.9 > tau and the logit leaves the row's denominator.
@pytest.mark.parametrize("dtype,margin,m", [("bf16", "arcface", 0.5), ("f16", "cosface", 0.4)])
def test_conflict_filter(dev, dtype, margin, m):
    out = _case(dev, 300, 512, 20000, 0.1, dtype, margin, m, seed=14, tau=0.4, conflicts=3)
    assert out["n_filtered"] >= 50


def test_conflict_filter_ragged_and_unowned(dev):
    out = _case(dev, 100, 256, 5000, 0.2, "bf16", "arcface", 0.5, seed=15, class_offset=1000,
                label_span=(1000, 6500), tau=0.4, conflicts=2)
    assert out["n_filtered"] >= 20


def test_conflict_filter_fp32(dev):
    out = _case(dev, 64, 128, 2000, 0.1, "f32", "cosface", 0.4, seed=16, tau=0.4, conflicts=2)
    assert out["n_filtered"] >= 20


def test_conflict_filter_full_softmax(dev):
    """FC*-1.0: the filter at r = 1."""
    out = _case(dev, 64, 128, 2000, 1.0, "bf16", "arcface", 0.5, seed=17, tau=0.4, conflicts=2)
    assert out["K"] == 2000 and out["n_filtered"] >= 20


def test_tau_at_least_one_is_pfc(dev):
    """tau >= 1 runs the unfiltered kernels: bit-identical to no filter."""
    from _gpu_util import make_problem
    outs = []
    for tau in (None, 1.0):
        Xd, Wd, Md, Pd, Ld = make_problem(200, 256, 6000, "bf16", 18, device=dev, conflicts=2)
        shard = _shard(200, 256, 6000, 0.1, "bf16", "arcface", 0.5, dev=dev, tau=tau)
        shard.step(Xd, Ld, Wd, Md, 18)
        torch.cuda.synchronize()
        outs.append((shard.loss.clone(), shard.dX.clone(), Wd.clone(), Md.clone()))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


def _empty_row_problem(seed, dtype, dev, B=96, d=128, C=2000, a=1000, n_empty=3, mu=10.0):
    """Class centres sharing a common direction u, and a few rows along u whose
    labels lie outside the shard [a, a + C): every active cosine of such a row
    is ~0.66, above tau = 0.3, so the PFC* filter leaves its denominator empty.
    The other rows are ordinary Gaussian rows with owned labels."""
    rng = np.random.default_rng(seed)
    u = rng.standard_normal(d)
    u /= np.linalg.norm(u)
    W = (0.01 * (rng.standard_normal((C, d)) + mu * u)).astype(np.float32)
    X = rng.standard_normal((B, d)).astype(np.float32)
    labels = rng.integers(a, a + C, size=B)
    for k in range(n_empty):
        n = 7 + 31 * k
        X[n] = (np.sqrt(d) * u + 0.3 * rng.standard_normal(d)).astype(np.float32)
        labels[n] = a + C + 17 * k
    M = (1e-3 * rng.standard_normal((C, d))).astype(np.float32)
    t = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    return (torch.from_numpy(X).to(t).to(dev), torch.from_numpy(W).to(t).to(dev),
            torch.from_numpy(M).to(dev), None, torch.from_numpy(labels).to(dev))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_conflict_filter_empty_denominator(dev, dtype):
    """Rows whose label is outside the shard and whose every logit the PFC*
    filter drops: lse = -inf, no probability, no gradient, no NaN anywhere."""
    from _gpu_util import run_and_compare
    seed, tau = 32, 0.3
    print(f"\nempty-denominator rows: dtype={dtype} seed={seed} tau={tau}", flush=True)
    Xd, Wd, Md, Pd, Ld = _empty_row_problem(seed, dtype, dev)
    shard = _shard(96, 128, 2000, 0.2, dtype, "arcface", 0.5, class_offset=1000, dev=dev,
                   tau=tau)
    out = run_and_compare(shard, Xd, Wd, Md, Pd, Ld, seed, "arcface")
    print(out, flush=True)
    assert out["n_empty_rows"] == 3
    assert bool(torch.isfinite(Wd).all()) and bool(torch.isfinite(Md).all())
    empty = torch.isneginf(shard.row_lse)
    assert int(empty.sum()) == 3
    assert bool((shard.dX[empty] == 0).all())


@pytest.mark.parametrize("dtype,B", [("bf16", 60), ("f16", 60), ("bf16", 600), ("f32", 60)])
def test_only_the_target_is_live(dev, dtype, B):
    """A filter that drops every negative and a margin that puts the target's
    logit far below zero (CosFace m = 3: lse around -190): probability 1, no
    gradient, and no NaN from the 128-class groups without a live logit."""
    from _gpu_util import make_problem
    d, C = 128, 9000
    print(f"\nonly the target live: {dtype} B={B}", flush=True)
    Xd, Wd, Md, _, Ld = make_problem(B, d, C, dtype, 74, random_m=False, device=dev)
    shard = _shard(B, d, C, 1.0, dtype, "cosface", 3.0, dev=dev, tau=-2.0)
    W0 = Wd.clone()
    shard.step(Xd, Ld, Wd, Md, 74)
    torch.cuda.synchronize()
    # lse = f_y up to the rounding of a logarithm and an exponential near 2^8
    # (2^-16 and less), which is also the most by which p can miss 1.
    assert bool((shard.row_lse < -100).all())
    assert float(shard.loss.abs()) <= 1e-4
    assert float(shard.dX.abs().max()) <= 1e-3 and float(Md.abs().max()) <= 1e-2
    assert bool(torch.isfinite(Wd).all()) and float((Wd.float() - W0.float()).abs().max()) <= 2e-3


@pytest.mark.parametrize("d,dtype,margin,m,seed", [
    (512, "f16", "arcface", 0.5, 20),
    (256, "bf16", "cosface", 0.4, 22),
    (128, "bf16", "arcface", 0.5, 23),
])
def test_batch_at_limit_16bit(dev, d, dtype, margin, m, seed):
    """The largest batch the ABI accepts (PFC_MAX_BATCH = 8192) at each feature
    width of the 16-bit path; the positives (~7,400 distinct labels) nearly
    fill the budget of 8,000."""
    from paper_2010_05222_amd import pfc
    assert pfc.PFC_MAX_BATCH == 8192
    out = _case(dev, 8192, d, 40000, 0.2, dtype, margin, m, seed=seed, random_m=False)
    assert out["K"] == 8000


def test_batch_at_limit_fp32(dev):
    """The largest batch of the fp32 path (4096 rows); here |P| > b, so S = P."""
    out = _case(dev, 4096, 128, 3000, 0.5, "f32", "cosface", 0.4, seed=21)
    assert out["K"] == out["n_pos"] > 1500


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_mapped_label_past_active_set_is_unowned(dev, dtype):
    """A labels_mapped entry at or past |S| (never produced by the sampler,
    but accepted by the forward and backward calls) counts as an unowned
    label: no target term and a zero loss term, as the oracle computes for a
    label of -1.  The id list is valid past |S| here, so the call reads no
    out-of-range class either way."""
    from _gpu_util import make_problem, row_rel_err, MAX_ABS, REL_ROW
    B, d, C, r, seed = 200, 128, 1000, 0.05, 41
    labels = np.random.default_rng(41).integers(0, 30, size=B)   # 30 classes: |S| = 50 < cap
    print(f"\ncase B={B} d={d} C={C} r={r} dtype={dtype} seed={seed} mapped label past |S|",
          flush=True)
    Xd, Wd, Md, Pd, Ld = make_problem(B, d, C, dtype, seed, labels=labels, device=dev)
    shard = _shard(B, d, C, r, dtype, "arcface", 0.5, 0, dev)
    X64 = Xd.double().cpu().numpy()
    W0 = Wd.double().cpu().numpy()
    M0 = Md.double().cpu().numpy()
    shard.sample(Ld, seed)
    torch.cuda.synchronize()
    K = int(shard.n_active.item())
    assert K + 5 < shard.cap, (K, shard.cap)
    shard.active[K + 5] = 0
    row = 7
    shard.labels_mapped[row] = K + 5
    shard.forward(Xd, Wd)
    shard.backward(Xd, Wd, Md, None)
    torch.cuda.synchronize()

    active = shard.active[:K].cpu().numpy()
    mapped = shard.labels_mapped.cpu().numpy().copy()
    mapped[row] = -1
    Ws = W0[active]
    fw = O.forward(X64, Ws, mapped, shard.s, shard.m, "arcface")
    loss_ref = O.batch_loss(fw["row_loss"], B)
    dx_ref = O.grad_x(X64, Ws, mapped, fw["lse"], B, shard.s, shard.m, "arcface")
    g_ref = O.grad_w(X64, Ws, np.arange(K), mapped, fw["lse"], B, shard.s, shard.m, "arcface")
    loss = float(shard.loss.item())
    dx = shard.dX.cpu().numpy().astype(np.float64)
    g = Md.double().cpu().numpy()[active] - shard.mu * M0[active]
    assert abs(loss - loss_ref) <= 1e-3 * abs(loss_ref), (loss, loss_ref)
    assert np.max(np.abs(dx - dx_ref)) <= MAX_ABS[dtype]
    assert np.max(row_rel_err(dx, dx_ref)) <= REL_ROW[dtype]
    assert np.max(np.abs(g - g_ref)) <= MAX_ABS[dtype]


def test_pipeline_equals_serial_steps(dev):
    """PfcPipeline (each step's active set drawn on a side stream beside the
    previous step) gives the serial steps' loss, row_lse, dX, W and momentum
    bit for bit over four steps with different batches and seeds."""
    from paper_2010_05222_amd.head import PfcPipeline
    from _gpu_util import make_problem
    B, d, C, r, T = 96, 256, 5000, 0.1, 4
    print(f"\ncase B={B} d={d} C={C} r={r} bf16 pipeline vs serial, {T} steps", flush=True)
    Xd, Wd, Md, _, _ = make_problem(B, d, C, "bf16", 51, device=dev)
    rng = np.random.default_rng(52)
    Ls = [torch.from_numpy(rng.integers(0, C, size=B)).to(dev) for _ in range(T)]
    Xs = [torch.roll(Xd, 7 * t, 0).contiguous() for t in range(T)]
    W1, M1, W2, M2 = Wd.clone(), Md.clone(), Wd.clone(), Md.clone()
    shard = _shard(B, d, C, r, "bf16", "arcface", 0.5, 0, dev)
    serial = []
    for t in range(T):
        shard.step(Xs[t], Ls[t], W1, M1, 100 + t)
        serial.append((shard.loss.clone(), shard.row_lse.clone(), shard.dX.clone()))
    pipe = PfcPipeline(B, d, C, r, dtype="bf16", s=64.0, m=0.5, margin="arcface", lr=0.1,
                       mu=0.9, device=dev)
    pipe.begin(Ls[0], 100)
    for t in range(T):
        last = t + 1 == T
        out = pipe.step(Xs[t], W2, M2, None if last else Ls[t + 1], None if last else 101 + t)
        got = (out.loss.clone(), out.row_lse.clone(), out.dX.clone())
        for a, b in zip(got, serial[t]):
            assert torch.equal(a, b), t
    torch.cuda.synchronize()
    assert torch.equal(W1, W2) and torch.equal(M1, M2)
    with pytest.raises(RuntimeError):
        pipe.step(Xs[0], W2, M2)          # no active set drawn for a fifth step
