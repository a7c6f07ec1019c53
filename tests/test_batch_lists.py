"""Which batched chains list their movable tasks: large ones with bit-serial
decisions only, since the list costs a chain of few tasks, or of one-bit
decisions, more than it saves (up to twice the time)."""
import kernel_resources as kr
from plan_helpers import plans  # noqa: F401  (fixture)


# (tasks, threads): chains that listing was measured to help, and to slow down
HELPED = [(2048, 256), (2048, 512), (2048, 1024), (1600, 1024), (900, 256), (900, 512), (771, 256), (771, 512),
          (300, 256), (400, 256)]
SLOWED = [(32, 256), (32, 1024), (100, 256), (100, 512), (300, 512), (300, 1024), (400, 512), (512, 256), (512, 512),
          (512, 1024)]


def test_rule(plans):
    def lists(one_bit, metro, cases):
        return [a == "1" for a in plans(["batch %d %d %d %d" % ((one_bit, metro) + c) for c in cases])]
    for metro in (0, 1):
        assert all(lists(0, metro, HELPED))
        assert not any(lists(0, metro, SLOWED))
        assert not any(lists(1, metro, HELPED + SLOWED))
    # one pass of more than 8 wavefronts
    assert all(lists(0, 0, [(771, 1024), (900, 1024)])) and not any(lists(0, 1, [(771, 1024), (900, 1024)]))


def test_kernels_without_lists_hold_none():
    """The batch kernels that list nothing keep the LDS they need to share a CU."""
    ks = {n: k for n, k in kr.kernels().items() if "domino_batch_kernelI" in n and "ELb0EE" in n}
    assert len(ks) == 6 and sum("domino_batch_kernelILi2" in n for n in ks) == 2
    for name, k in ks.items():
        assert k[".group_segment_fixed_size"] <= 256, name


def test_resident_work_groups(plans):
    """The work-groups counted per CU fit it with the kernels' own static LDS, and
    one more would not."""
    static = {lists: {k[".group_segment_fixed_size"] for n, k in kr.kernels().items()
                      if "domino_batch_kernelI" in n and ("ELb1EE" if lists else "ELb0EE") in n} for lists in (0, 1)}
    cases = [(64 * n * -(-n // 128), lists, threads) for n in range(1, 513) for threads in (64, 256, 512, 1024)
             for lists in (0, 1)]
    for (state, lists, threads), got in zip(cases, plans(["batch_lds %d %d %d" % c for c in cases])):
        s, per_cu = map(int, got.split())
        assert {s} == static[lists]
        assert 1 <= per_cu <= 2048 // threads and per_cu * (state + s) <= kr.LDS_BYTES
        assert per_cu == 2048 // threads or (per_cu + 1) * (state + s) > kr.LDS_BYTES
