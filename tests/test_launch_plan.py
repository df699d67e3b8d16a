"""The schedule a call takes on the host: the ABI layer (csrc/api.cpp) with stubs of the kernel launchers, compiled
with g++ into a small program that prints what each call would launch (no GPU).

Long sequences in grids of more than one dispatch round (256 workgroups) are cut at 2048 positions if the workspace
holds the partials: from 8192 positions in up to 320 (layer, sequence, KV head) groups, from 10240 in up to 352, and
where a call has policies per layer from 8192 in up to 512 groups and from 3072 in more.  Every other automatic call
of such a grid keeps its groups whole, with any workspace."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_01483_amd", "csrc")
OK, ENOSPACE = 0, -3

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

DRIVER = r"""
#include <stdio.h>
#include <string.h>
#include "internal.h"
using namespace murmur;
static AttnLaunch got;
namespace murmur {
int launch_evict_compact(const murmur_seg *, const murmur_policy *, int32_t, int32_t, int32_t *, int32_t, int32_t *,
                         int32_t *, const int32_t *, int32_t, int32_t, murmur_stream_t) { return 0; }
int launch_decode_attn(const AttnLaunch &a, murmur_stream_t) { got = a; return 0; }
int launch_workspace_init(int32_t *, int64_t, murmur_stream_t) { return 0; }
int launch_read_probe(const void *, int64_t, int32_t, int32_t, int32_t, bool, uint32_t *, murmur_stream_t) { return 0; }
int launch_paged_step(const murmur_seg *, const murmur_policy *, int32_t, int32_t, int32_t *, int32_t, int32_t,
                      int32_t *, int32_t *, int32_t, int32_t, murmur_stream_t) { return 0; }
int launch_paged_append(const murmur_seg *, int32_t, const int32_t *, int32_t, int32_t, const murmur_kv &, int32_t,
                        const void *, const void *, murmur_stream_t) { return 0; }
int static_scratch(void **p, bool *fresh) { *p = (void *)0x100000; *fresh = false; return 0; }
int read_and_clear_device_error(murmur_stream_t, int32_t *) { return 0; }
const char *hip_error_text(int) { return "stub"; }
}  // namespace murmur
int main() {  // lines: call mode layers batch Hq Hkv max_keep split_len ws_bytes (-1: what the workspace query says)
    void *f = (void *)0x100000;
    int32_t *fi = (int32_t *)f;
    char call[16];
    int mode, nl, b, hq, hkv, keep, split;
    long long ws;
    while (scanf("%15s %d %d %d %d %d %d %d %lld", call, &mode, &nl, &b, &hq, &hkv, &keep, &split, &ws) == 9) {
        size_t need = 0;
        murmur_decode_attn_workspace(nl, b, hq, hkv, keep, split, &need);
        const size_t bytes = ws < 0 ? need : (size_t)ws;
        murmur_kv kv{f, f, nl, 1 << 20, 1LL << 40, 1LL << 32, 1LL << 28, 128};
        const murmur_seg *seg = (const murmur_seg *)f;
        const murmur_policy *pol = (const murmur_policy *)f;
        const murmur_ring ring{64, f, f};
        got = AttnLaunch{};
        int rc = -1;
        if (!strcmp(call, "step"))
            rc = murmur_decode_step(seg, pol, mode, f, &kv, nullptr, nullptr, nullptr, keep, b, hq, hkv, 128, 1.f,
                                    split, f, 1, nullptr, f, bytes, nullptr);
        else if (!strcmp(call, "static"))
            rc = murmur_decode_step_static(seg, pol, mode, f, &kv, nullptr, nullptr, nullptr, keep, b, hq, hkv, 128,
                                           1.f, split, f, 1, nullptr, nullptr);
        else if (!strcmp(call, "ring"))
            rc = murmur_decode_step_ring(seg, pol, mode, &ring, f, &kv, nullptr, nullptr, nullptr, keep, b, hq, hkv,
                                         128, 1.f, split, f, 1, nullptr, f, bytes, nullptr);
        else if (!strcmp(call, "ranges"))
            rc = murmur_decode_attn(f, &kv, nullptr, fi, nullptr, keep, b, hq, hkv, 128, 1.f, split, f, 1, nullptr, f,
                                    bytes, nullptr);
        else if (!strcmp(call, "index"))
            rc = murmur_decode_attn(f, &kv, fi, nullptr, fi, keep, b, hq, hkv, 128, 1.f, split, f, 1, nullptr, f,
                                    bytes, nullptr);
        printf("%d %d %d %zu %d\n", rc, got.n_split, got.split_len, need, got.stream_count);
    }
    return 0;
}
"""

PER_SEQ, PER_LAYER = 1, 2


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "driver.cpp", d / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{ROOT}/include", f"-I{CSRC}", str(src),
                    os.path.join(CSRC, "api.cpp"), "-o", str(exe)], check=True, capture_output=True, text=True)

    def run(call, mode, nl, b, keep, hq=28, hkv=4, split=0, ws=-1, stream=False):
        """(status, splits, split length, bytes the workspace query returns), or with `stream` the retained count
        from which a sequence's K/V rows are streamed"""
        line = f"{call} {mode} {nl} {b} {hq} {hkv} {keep} {split} {ws}\n"
        out = subprocess.run([str(exe)], input=line, capture_output=True, text=True, check=True).stdout
        got = tuple(int(x) for x in out.split())
        return got[4] if stream else got[:4]

    return run


ONE_POLICY = pytest.mark.parametrize("call,mode", [("step", 0), ("step", PER_SEQ), ("ring", PER_SEQ), ("ranges", 0),
                                                   ("index", 0)])


@ONE_POLICY
@pytest.mark.parametrize("nl,b", [(28, 12), (14, 12), (28, 6), (28, 4), (32, 3), (1, 89)])
def test_groups_of_one_policy_stay_whole(plan, call, mode, nl, b):
    for keep in (2600, 3071, 3072, 3200, 4096, 8191, 8192, 20000):
        for ws in (-1, 256, 1 << 30):
            assert plan(call, mode, nl, b, keep, ws=ws)[:2] == (OK, 1), (keep, ws)


def check_cut(plan, call, mode, nl, b, line):
    assert plan(call, mode, nl, b, line - 1)[:2] == (OK, 1)
    for keep in (line, line + 1, line + 2048):
        rc, n, split, need = plan(call, mode, nl, b, keep)
        assert (rc, n, split) == (OK, -(-keep // 2048), 2048)
        # a workspace that cannot hold the partials: the groups stay whole
        assert plan(call, mode, nl, b, keep, ws=need - 1)[:2] == (OK, 1)
        assert plan(call, mode, nl, b, keep, ws=256)[:2] == (OK, 1)
        assert plan(call, mode, nl, b, keep, ws=255)[0] == ENOSPACE
        assert plan(call, mode, nl, b, keep, ws=need + 12345)[:2] == (OK, n)
        assert n * nl * b * 4 * 7 * 130 * 4 <= 64 << 20 and need <= 74 << 20


@ONE_POLICY
@pytest.mark.parametrize("nl,b,line", [(13, 5, 8192), (20, 4, 8192), (27, 3, 10240), (28, 3, 10240), (22, 4, 10240)])
def test_long_sequences_are_cut_in_little_more_than_a_round(plan, call, mode, nl, b, line):
    check_cut(plan, call, mode, nl, b, line)


@pytest.mark.parametrize("call", ["step", "ring"])
@pytest.mark.parametrize("mode", [PER_LAYER, PER_LAYER | PER_SEQ])
def test_long_sequences_are_cut_with_policies_per_layer(plan, call, mode):
    for nl, b, line in ((28, 12, 3072), (14, 12, 3072), (43, 3, 3072), (32, 4, 8192), (28, 4, 8192), (28, 3, 8192),
                        (13, 5, 8192)):
        check_cut(plan, call, mode, nl, b, line)
    # partials beyond 64 MiB: whole, and no workspace asked for
    assert plan(call, mode, 28, 12, 35000)[:2] == (OK, 1) and plan(call, mode, 28, 12, 35000)[3] == 256
    # one dispatch round: the same splits as with one policy
    for keep in (850, 3200, 9000, 35000):
        assert plan(call, mode, 2, 12, keep) == plan(call, PER_SEQ, 2, 12, keep)


def test_static_step_takes_what_its_scratch_holds(plan):
    assert plan("static", PER_SEQ, 28, 12, 3200)[:2] == (OK, 1)
    assert plan("static", PER_LAYER, 28, 12, 3200)[:2] == (OK, 1)   # 11 MiB of partials and tickets: whole
    rc, n, split, need = plan("static", PER_LAYER, 13, 5, 8192, hq=4, hkv=4)
    assert need <= 4 << 20 and (rc, n, split) == (OK, 4, 2048)
    assert plan("static", PER_LAYER, 28, 12, 1024, split=512)[0] == ENOSPACE  # an explicit length is kept


@pytest.mark.parametrize("call", ["step", "ring", "ranges", "index"])
def test_explicit_splits_need_their_workspace(plan, call):
    rc, n, split, need = plan(call, PER_SEQ, 28, 12, 4096, split=2048)
    assert (rc, n, split) == (OK, 2, 2048)
    assert plan(call, PER_SEQ, 28, 12, 4096, split=2048, ws=need - 1)[0] == ENOSPACE


@pytest.mark.parametrize("b,hkv,count", [(1, 4, 6144), (12, 4, 512), (64, 4, 96), (3, 1, 8192), (5, 4, 1229),
                                         (65535, 4, 1)])
def test_streaming_starts_at_twelve_mib_a_layer(plan, b, hkv, count):
    """The smallest count with b * hkv * count * 512 bytes of K and V at 12 MiB or more."""
    assert -(-(12 << 20) // (b * hkv * 512)) == count
    for call in ("step", "ring", "ranges", "index"):
        assert plan(call, 0, 1, b, 100, hq=hkv, hkv=hkv, stream=True) == count
