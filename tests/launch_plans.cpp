// Host check of the launch plans of erase_api.cpp, for random networks: no GPU,
// no HIP call.  The dispatcher is compiled in; the launchers are not needed.
//  * Every launch of every schedule has a tile, split and kind that the
//    launchers take.
//  * The blocks that share a launch agree on everything the host takes from
//    the first of them (kernel, grid, slices): the rest each block reads from
//    its own arguments.
// Arguments: seed, networks, then fixed networks as text (see parse()).
#include "erase_api.cpp"

#include <cstdlib>
#include <random>
#include <sstream>

namespace erase {
int xcd_group(int, int, int, int, int) { return 1; }
hipError_t launch_prologue(int, const PrologueArgs&, hipStream_t, const LaunchEv&) { return hipSuccess; }
hipError_t launch_gemm(int, int, const GemmDesc&, const EpiParams&, hipStream_t, const LaunchEv&, const Batch*) {
  return hipSuccess;
}
hipError_t launch_bwd_gemm(int, const GemmDesc&, const EpiParams&, const GemmDesc&, const EpiParams&, hipStream_t,
                           const LaunchEv&, const Batch*) {
  return hipSuccess;
}
hipError_t launch_head(int, const HeadArgs&, hipStream_t, const LaunchEv&, const Batch*) { return hipSuccess; }
hipError_t launch_adam(int, const AdamArgs&, hipStream_t, const LaunchEv&, const Batch*) { return hipSuccess; }
hipError_t launch_wgrad_adam(int, const GemmDesc&, const EpiParams&, const AdamArgs&, hipStream_t, const LaunchEv&,
                             const Batch*) {
  return hipSuccess;
}
hipError_t launch_refresh(int, const AdamArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_embed_bags(int, const EmbedArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_embed_bags_backward(int, const EmbedBwdArgs&, hipStream_t) { return hipSuccess; }
hipError_t bag_scratch_device_ptr(void**, size_t*) { return hipSuccess; }
}  // namespace erase

namespace {

struct Net {
  erase_config c{};
  std::vector<erase_block_spec> blocks;
  std::vector<std::vector<erase_layer_spec>> layers;
};

erase_layer_spec layer(int kind, int in, int out) {
  erase_layer_spec s{};
  s.kind = kind;
  s.in_dim = in;
  s.out_dim = out;
  return s;
}

void finish(Net& n) {
  n.blocks.resize(n.layers.size());
  for (size_t b = 0; b < n.layers.size(); ++b) {
    n.blocks[b].layers = n.layers[b].data();
    n.blocks[b].n_layers = (int)n.layers[b].size();
    n.blocks[b].loss = ERASE_LOSS_BCE;
    n.blocks[b].lambda = 1.f;
  }
  n.c.blocks = n.blocks.data();
  n.c.n_blocks = (int)n.blocks.size();
  n.c.x_ld = (int)roundup(n.c.in_dim, 128);
  n.c.x_in_place = n.c.batch % 128 == 0;
  n.c.lr = 1e-3f;
  n.c.beta1 = 0.9f;
  n.c.beta2 = 0.999f;
  n.c.eps = 1e-8f;
}

// "bf16 4096 512 x:6:c0:512,512" = dtype, batch, input width, then runs of
// blocks: source, count, cross layers, widths
Net parse(const std::string& text) {
  Net n;
  std::istringstream in(text);
  std::string dt, run;
  in >> dt >> n.c.batch >> n.c.in_dim;
  n.c.dtype = dt == "f32" ? ERASE_F32 : ERASE_BF16;
  int cur = n.c.in_dim;
  std::vector<int> src;
  while (in >> run) {
    std::replace(run.begin(), run.end(), ':', ' ');
    std::replace(run.begin(), run.end(), ',', ' ');
    std::istringstream r(run);
    std::string s, cross;
    int count, w;
    r >> s >> count >> cross;
    std::vector<int> widths;
    while (r >> w) widths.push_back(w);
    for (int i = 0; i < count; ++i) {
      const bool prev = s == "p";
      int k = prev ? cur : n.c.in_dim;
      std::vector<erase_layer_spec> ls;
      for (int x = 0; x < std::atoi(cross.c_str() + 1); ++x) ls.push_back(layer(ERASE_LAYER_CROSS, k, k));
      for (int o : widths) {
        ls.push_back(layer(ERASE_LAYER_LINEAR_RELU, k, o));
        k = o;
      }
      cur = k;
      n.layers.push_back(ls);
      src.push_back(prev ? ERASE_IN_PREV : ERASE_IN_X);
    }
  }
  finish(n);
  for (size_t b = 0; b < src.size(); ++b) n.blocks[b].input_src = src[b];
  return n;
}

// runs of equal blocks, on x or chained, widths up to 2048, 1 to 40 blocks
std::string random_net(std::mt19937& g) {
  auto uni = [&](int a, int b) { return a + (int)(g() % (unsigned)(b - a + 1)); };
  auto logi = [&](double a, double b) {
    return (int)std::lround(std::exp(std::log(a) + (std::log(b) - std::log(a)) * (g() / 4294967296.0)));
  };
  std::ostringstream o;
  int batch = logi(32, 32768);
  if (uni(0, 1)) batch = (int)roundup(batch, 128);
  const int in = logi(16, 2048);
  o << (uni(0, 4) ? "bf16 " : "f32 ") << batch << ' ' << in;
  int left = uni(0, 2) ? uni(1, 12) : uni(1, 40), cur = in;
  bool first = true;
  while (left > 0) {
    const bool prev = !first && uni(0, 1);
    int count = std::min(left, uni(0, 2) ? left : uni(1, left));
    const int L = uni(1, 3), cross = uni(0, 3) ? 0 : uni(1, 2);
    std::vector<int> w;
    for (int l = 0; l < L; ++l) w.push_back(logi(16, 2048));
    if (prev || uni(0, 2) == 0) w.back() = prev ? cur : in;  // a chain of equal blocks needs equal ends
    o << ' ' << (prev ? 'p' : 'x') << ':' << count << ":c" << cross << ':';
    for (int l = 0; l < L; ++l) o << (l ? "," : "") << w[l];
    cur = w.back();
    left -= count;
    first = false;
  }
  return o.str();
}

std::string describe(const Op& o) {
  std::ostringstream s;
  auto gd = [&](const GemmDesc& g) {
    s << " [" << g.M << "x" << g.N << "x" << g.K << " tile " << g.bm << "x" << g.bn << " split " << g.split << " kps "
      << g.kps << " kg " << g.kgroups << "]";
  };
  s << "type " << o.type << " kind " << o.kind << " layer " << o.layer << " slot " << o.slot;
  gd(o.j.g);
  gd(o.j.g2);
  s << " chunks " << o.j.a.nchunks << " rows " << o.j.h.rows << " fused " << (o.j.e.ap != nullptr);
  return s.str();
}

// Everything launch_op and the launchers take from the first block.
bool agree(const Op& a, const Op& b) {
  auto gd = [](const GemmDesc& x, const GemmDesc& y) {
    return x.M == y.M && x.N == y.N && x.K == y.K && x.kps == y.kps && x.split == y.split && x.bm == y.bm &&
           x.bn == y.bn && x.kgroups == y.kgroups && x.lda == y.lda && x.ldb == y.ldb;
  };
  return a.type == b.type && a.kind == b.kind && a.layer == b.layer && a.slot == b.slot && gd(a.j.g, b.j.g) &&
         gd(a.j.g2, b.j.g2) && (a.j.e.ap != nullptr) == (b.j.e.ap != nullptr) && a.j.a.nchunks == b.j.a.nchunks &&
         a.j.a.nseg == b.j.a.nseg && a.j.a.nloss == b.j.a.nloss && a.j.h.M == b.j.h.M && a.j.h.N == b.j.h.N &&
         a.j.h.rows == b.j.h.rows && (a.j.h.dmn != nullptr) == (b.j.h.dmn != nullptr);
}

// The forms the launchers have.
bool gemm_taken(int bf, int kind, const GemmDesc& g, const EpiParams& e) {
  const int BK = bf ? 64 : 32;
  if (g.K % BK || g.kps % BK || g.kps <= 0 || int64_t(g.split) * g.kps < g.K || int64_t(g.split - 1) * g.kps >= g.K)
    return false;
  if (kind != GK_WGRAD && g.split != 1) return false;
  if (e.ap && !(kind == GK_WGRAD && g.bm == 64 && g.bn == 64 && g.kgroups == 2 && g.split == 1)) return false;
  const bool fwd = kind == GK_FWD_RELU || kind == GK_FWD_CROSS, other = kind == GK_DGRAD || kind == GK_WGRAD;
  if (bf && kind == GK_FWD_HEAD) return g.bm == 16 && g.N <= 128;
  if (bf && (g.bm == 256 || g.bm == 128)) return g.bn == g.bm && (fwd || other);
  if (bf && g.bm == 64 && g.bn == 128) return fwd && g.kgroups == 2;
  if (g.bm != 64 || g.bn != 64) return false;
  if (g.kgroups == 2) return kind == GK_WGRAD ? g.split == 1 && (!bf || e.ap) : bf && fwd;
  return fwd || other || (kind == GK_FWD_HEAD && g.N <= 64);
}
bool taken(int bf, const Op& o) {
  const GemmDesc &g = o.j.g, &w = o.j.g2;
  switch (o.type) {
    case Op::GEMM: return gemm_taken(bf, o.kind, g, o.j.e);
    case Op::PAIR:
      return g.bm == w.bm && g.bn == w.bn && g.bm == g.bn && g.split == 1 && !o.j.e2.ap && g.kps >= g.K &&
             gemm_taken(bf, GK_DGRAD, g, o.j.e) && gemm_taken(bf, GK_WGRAD, w, o.j.e2);
    case Op::WGRAD_ADAM: return o.j.e.ap && gemm_taken(bf, GK_WGRAD, g, o.j.e);
    case Op::HEAD: return o.j.h.N >= 1 && o.j.h.N <= HEAD_MAX_N && o.j.h.rows >= 1;
    default: return o.j.a.nchunks > 0;
  }
}

int check(const std::string& text) {
  Net n = parse(text);
  if (validate(&n.c, nullptr) != ERASE_OK) return -1;
  Ctx c;
  c.cfg = n.c;
  build_plan(c.cfg, 4096, &c.P);
  std::vector<erase_block_buffers> bufs(n.c.n_blocks);
  for (auto& b : bufs) b.param = b.m = b.v = b.grad = reinterpret_cast<float*>(uintptr_t(4096));
  build_segments(&c.P, bufs.data());
  StepIn in;
  in.x = kStepX;
  in.ldx = c.P.x_in_place ? c.cfg.x_ld : c.P.ldxp;
  in.p = {kStepX, nullptr, nullptr, nullptr};
  auto ops = [&](int b, bool send) {
    std::vector<Op> v;
    auto put = [&](Op& o) {
      v.push_back(o);
      return ERASE_OK;
    };
    (void)forward_ops(&c, b, in, true, 0, c.P.blk[b].L, put);
    (void)backward_ops(&c, b, in, send, true, put);
    (void)backward_ops(&c, b, in, send, false, put);
    (void)head_op(&c, b, in, put);
    (void)adam_op(&c, b, in, put);
    return v;
  };
  int bad = 0;
  for (int b = 0; b < n.c.n_blocks; ++b)
    for (int send = 0; send < (c.P.undet_ok ? 2 : 1); ++send)
      for (const Op& o : ops(b, send))
        if (!taken(c.P.bf16, o)) {
          std::printf("not taken (%s): block %d undetached %d: %s\n", text.c_str(), b, send, describe(o).c_str());
          ++bad;
        }
  for_each_unit(&c.P, [&](Unit& u) {
    for (const Group& g : u.groups) {
      const std::vector<Op> a = ops(g.first, false);
      for (int i = 1; i < g.n; ++i) {
        const std::vector<Op> v = ops(g.first + i, false);
        bool ok = v.size() == a.size();
        for (size_t k = 0; ok && k < v.size(); ++k)
          if (!agree(a[k], v[k])) {
            std::printf("differ (%s), unit of %d: block %d: %s\n  block %d: %s\n", text.c_str(), u.n, g.first,
                        describe(a[k]).c_str(), g.first + i, describe(v[k]).c_str());
            ok = false;
          }
        bad += ok ? 0 : 1;
      }
    }
  });
  return bad;
}

}  // namespace

int main(int argc, char** argv) {
  const int seed = std::atoi(argv[1]), count = std::atoi(argv[2]);
  std::mt19937 g(seed);
  int bad = 0, nets = 0, badnets = 0;
  auto one = [&](const std::string& t) {
    const int r = check(t);
    if (r < 0) return false;
    ++nets;
    bad += r;
    badnets += r > 0;
    return true;
  };
  for (int i = 3; i < argc; ++i)
    if (!one(argv[i])) std::printf("refused: %s\n", argv[i]), ++bad;
  for (int i = 0; i < count;) i += one(random_net(g)) ? 1 : 0;
  std::printf("%d networks, %d with faults, %d faults\n", nets, badnets, bad);
  return bad != 0;
}
